// F32 instantiation of the hop for small launches.
#include "hop_small.h"

namespace mspcg {

template int launch_hop_small<F32>(const HopArgs<F32>&, int, int, bool, hipStream_t);

}  // namespace mspcg

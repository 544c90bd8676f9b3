// F64 instantiation of the hop for small launches.
#include "hop_small.h"

namespace mspcg {

template int launch_hop_small<F64>(const HopArgs<F64>&, int, int, bool, hipStream_t);

}  // namespace mspcg

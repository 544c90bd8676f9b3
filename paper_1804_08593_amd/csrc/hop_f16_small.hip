// F16 instantiation of the hop for small launches.
#include "hop_small.h"

namespace mspcg {

template int launch_hop_small<F16>(const HopArgs<F16>&, int, int, bool, hipStream_t);

}  // namespace mspcg

// F64 instantiation of the Ls-vectorised hop (one translation unit per
// storage precision so the kernels compile in parallel).
#include "hop_impl.h"

namespace mspcg {

MSPCG_HOP_WIDE(MSPCG_HOP_EXTERN, F64)

template int launch_hop<F64>(const HopArgs<F64>&, int, int, bool, bool, hipStream_t,
                             const HopReach*);
template int launch_multi_hop<F64>(const MultiHop<F64>*, long, int, bool, bool, bool,
                                    bool, hipStream_t);

}  // namespace mspcg

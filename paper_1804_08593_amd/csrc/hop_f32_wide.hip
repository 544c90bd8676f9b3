// F32 instantiation of the hop kernels for the larger Ls.
#include "hop_impl.h"

namespace mspcg {

MSPCG_HOP_WIDE(MSPCG_HOP_INST, F32)

}  // namespace mspcg

// The FP16 block hop on the matrix cores (hop_rows.h).
#include <string.h>

#include "hop_rows.h"

namespace mspcg {

namespace {

template <bool DAG, bool INV>
__global__ __launch_bounds__(kRowWaves * 64, 3) void row_kernel(RowArgs a) {
    if (a.done && *a.done) return;
    int bx, d;
    logical_block(a.xcd_remap, bx, d);
    rows::row_body<DAG, INV>((const RowArgs*)__builtin_amdgcn_kernarg_segment_ptr(), bx, d,
                               (int)gridDim.x);
}

}  // namespace

int launch_hop_rows(const HopArgs<F16>& h, int Ls, int ndom, bool dag, const HopReach& reach,
                    hipStream_t st) {
    RowArgs a;
    memset(&a, 0, sizeof(a));
    a.in = h.in;
    a.out = h.out;
    a.aux = h.aux;
    a.links = h.links;
    a.link_dom_stride = h.link_dom_stride;
    a.g = h.g;
    a.has_aux = h.has_aux;
    a.partials = h.partials;
    a.done = h.done;
    a.xcd_remap = h.xcd_remap;
    a.chunk = row_chunk(h.g.out, ndom);
    a.reach = reach.dist;
    for (int m = 0; m < 4; ++m) a.blk[m] = reach.blk[m];
    if (Ls != rows::LS || h.cg_r.data) return -1;
    // the block operator's programs have the form that RowProg holds, and an
    // inverse step only without aux, partials and update
    if (!row_prog_of(h.ph, dag, h.mf, Ls, a.rh)) return -1;
    if (h.has_aux && (!row_prog_of(h.pa, dag, h.mf, Ls, a.ra) || a.ra.inv)) return -1;
    if (a.rh.inv && (h.has_aux || h.partials)) return -1;
    const dim3 grid((unsigned)row_grid_x(h.g.out, ndom), (unsigned)ndom), block(kRowWaves * 64);
#define MSPCG_ROW_LAUNCH(D, I) hipLaunchKernelGGL((row_kernel<D, I>), grid, block, 0, st, a)
    if (dag && a.rh.inv) MSPCG_ROW_LAUNCH(true, true);
    else if (dag) MSPCG_ROW_LAUNCH(true, false);
    else if (a.rh.inv) MSPCG_ROW_LAUNCH(false, true);
    else MSPCG_ROW_LAUNCH(false, false);
#undef MSPCG_ROW_LAUNCH
    return 0;
}

}  // namespace mspcg

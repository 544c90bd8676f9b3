// The FP16 block hop on the matrix cores (hop_rows.h).
#include <string.h>

#include "hop_rows.h"

namespace mspcg {

namespace {

template <bool DAG, bool INV, int CG>
__global__ __launch_bounds__(kRowWaves * 64, 3) void row_kernel(RowArgs a) {
    if (a.done && *a.done) return;
    int bx, d;
    logical_block(a.xcd_remap, bx, d);
    rows::row_body<DAG, INV, CG>((const RowArgs*)__builtin_amdgcn_kernarg_segment_ptr(), bx, d,
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
    a.cg_r = h.cg_r;
    a.cg_x = h.cg_x;
    a.cg_p = h.cg_p;
    a.cg_sc = h.cg_sc;
    a.cg_alpha = h.cg_alpha;
    a.cg_first = h.cg_first;
    a.chunk = row_chunk(h.g.out, ndom);
    a.reach = reach.dist;
    for (int m = 0; m < 4; ++m) a.blk[m] = reach.blk[m];
    if (Ls != rows::LS || (h.cg_r.data && !dag)) return -1;
    // the block operator's programs have the form that RowProg holds, and an
    // inverse step only without aux, partials and update
    if (!row_prog_of(h.ph, dag, h.mf, Ls, a.rh)) return -1;
    if (h.has_aux && (!row_prog_of(h.pa, dag, h.mf, Ls, a.ra) || a.ra.inv)) return -1;
    if (h.cg_r.data && h.cg_keep_out) return -1;
    if (a.rh.inv && (h.has_aux || h.partials || h.cg_r.data)) return -1;
    const dim3 grid((unsigned)row_grid_x(h.g.out, ndom), (unsigned)ndom), block(kRowWaves * 64);
#define MSPCG_ROW_LAUNCH(D, I, C) \
    hipLaunchKernelGGL((row_kernel<D, I, C>), grid, block, 0, st, a)
    if (a.cg_x.data) MSPCG_ROW_LAUNCH(true, false, 2);
    else if (a.cg_r.data) MSPCG_ROW_LAUNCH(true, false, 1);
    else if (dag && a.rh.inv) MSPCG_ROW_LAUNCH(true, true, 0);
    else if (dag) MSPCG_ROW_LAUNCH(true, false, 0);
    else if (a.rh.inv) MSPCG_ROW_LAUNCH(false, true, 0);
    else MSPCG_ROW_LAUNCH(false, false, 0);
#undef MSPCG_ROW_LAUNCH
    return 0;
}

}  // namespace mspcg

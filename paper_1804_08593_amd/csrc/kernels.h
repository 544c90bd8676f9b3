// Kernel argument structures and host-side launchers of the MSPCG library.
#pragma once
#include "common.h"

// Fifth-dimension extents compiled into the kernels.
#define MSPCG_LS_LIST(X) X(2) X(4) X(6) X(8) X(10) X(12) X(16) X(20) X(24) X(32)

namespace mspcg {

// Geometry of one hop launch: every domain has an output box, an input box,
// an aux box and a link box (all relative to the domain origin).  The
// periodic (whole-lattice) case has one domain and four identical boxes.
struct HopGeom {
    Box out, in, aux, link;
    int out_par;   // global parity of the output sites
    int periodic;  // bit mu set: wrap at the input-box edges in direction mu (the
                   // box spans the lattice there); clear: drop hops leaving the box
};

struct DevScalars;

// Optional: the hop's result goes to a boundary field (complex128
// [Ls][V4][12], see mspcg.h) instead of `out`, with zeros on the sites of the
// other parity when zero_other.  Whole-lattice hops in FP64 and FP32 only; the
// FP16 block hops' arguments stay without it (a larger argument block slows them).
template <class S>
struct HopBoundary {
    double2* bout;
    long V4;
    int zero_other;
};
template <>
struct HopBoundary<F16> {};

template <class S>
struct HopArgs : HopBoundary<S> {
    CField<S> in;
    Field<S> out;
    CField<S> aux;
    const typename S::elem* links;
    long link_dom_stride;  // elements between the link arrays of consecutive domains
    HopGeom g;
    FiveDProg ph;  // applied to the hop result
    FiveDProg pa;  // applied to aux
    int has_aux;
    double mf;
    double* partials;  // optional: per (domain, workgroup) sum |out|^2
    const int* done;   // optional: skip the launch when *done != 0
    int xcd_remap;     // map workgroups so each XCD walks a contiguous site range
    int tile[4];       // nonzero: traverse output sites in 4D tiles of this extent
    // optional CG update fused after the output is formed (the last hop of A,
    // whole lattice or block domains):
    //   r -= alpha out ; x += alpha p (x = alpha p when cg_first; no x update
    //   when cg_x.data is null) ; partials = |r|^2 ; out is stored only when
    //   cg_keep_out.
    //   alpha is cg_alpha[domain] when given, else cg_sc->alpha.
    Field<S> cg_r;
    Field<S> cg_x;
    CField<S> cg_p;
    const DevScalars* cg_sc;
    const double* cg_alpha;
    int cg_keep_out;
    int cg_first;
    // optional: the output sites to compute, as checkerboard indices of the
    // output box shared by every domain (n_list of them); the traversal tile
    // is ignored then
    const int* site_list;
    long n_list;
};

// A FiveDProg as the FP16 matrix-core hop reads it, in single precision: with
// K (the plain hop) (1 - q K)^-1 then 1 + a K, with K^+ (the dagger hop) the
// reverse order, each where present.
struct RowProg {
    int bidi, inv;
    float a, corner;  // corner: -mf a
    float q, cinv;    // cinv: -mf / (1 + mf q^Ls)
    float su, sd;
};
// false: the program has a form that RowProg does not hold
inline bool row_prog_of(const FiveDProg& p, bool dag, double mf, int Ls, RowProg& r) {
    r = RowProg{};
    for (int k = 0; k < p.nsteps; ++k) {
        if ((p.dag[k] != 0) != dag) return false;
        if (p.kind[k] == STEP_BIDI) {
            if (r.bidi || (dag && r.inv)) return false;
            r.bidi = 1;
            r.a = (float)p.a[k];
            r.corner = (float)-(p.a[k] * mf);
        } else {
            if (r.inv || (!dag && r.bidi)) return false;
            r.inv = 1;
            double qL = 1;
            for (int s = 0; s < Ls; ++s) qL *= p.a[k];
            r.q = (float)p.a[k];
            r.cinv = (float)(-mf / (1.0 + mf * qL));
        }
    }
    r.su = (float)p.scale[0];
    r.sd = (float)p.scale[1];
    return true;
}

// Which of a block hop's output sites matter: those within `dist` sites (Manhattan
// distance) of the block of extent blk (0: not cut) at the domain origin; every one
// when dist < 0.
struct HopReach {
    long inner, widest;  // sites of the block and of the largest box of a domain
    int dist, blk[4];
};

// Arguments of the FP16 matrix-core hop (hop_rows.h), from HopArgs.
struct RowArgs {
    CField<F16> in, aux;
    Field<F16> out;
    const __half2* links;
    long link_dom_stride;
    HopGeom g;
    RowProg rh, ra;
    int has_aux, chunk, reach, blk[4], xcd_remap;
    double* partials;
    const int* done;
};

// x extent of a strip piece of the FP16 matrix-core hop (the last piece of a strip
// takes what is left, 2 at the least).  A piece loads two slices of inputs beyond its
// own, so pieces are cut no shorter than 4 where the box is that long; 6144 pieces are
// two rounds of the 3 waves per SIMD that its registers allow, so that the last round
// costs little.
inline int row_chunk(const Box& out, int ndom) {
    const long strips = (long)out.E[1] * out.E[2] * out.E[3] / 8 * ndom;
    int n = out.E[0];
    while (n > 4 && strips * ((out.E[0] + n - 1) / n) < 6144) n = (n / 2 + 1) & ~1;
    return n;
}

// small: hop_is_small launches take the small-launch kernel (hop_small.h); reach
// (FP16 block hops): hop_is_rows launches take the matrix-core kernel
template <class S>
int launch_hop(const HopArgs<S>& a, int Ls, int ndom, bool dag, bool small, hipStream_t st,
               const HopReach* reach = nullptr);
int launch_hop_rows(const HopArgs<F16>& a, int Ls, int ndom, bool dag, const HopReach& reach,
                    hipStream_t st);
template <class S>
int launch_hop_small(const HopArgs<S>& a, int Ls, int ndom, bool dag, hipStream_t st);

// Several lattices' block-domain hops of one stage in one persistent launch.
// The work list is (lattice i, domain d, workgroup bx): lattice i owns items
// [first[i], first[i+1]), ndom_i * gx[i] of them; a workgroup walks the list
// with a stride of the grid size and skips the items of lattices whose
// `done` flag (a[i].done) is set.  The lattices of one launch share Ls (8, 12
// or 16, multi_hop_ls) and the kernel variant (dagger, chain programs, fused
// update).  The descriptor lives in device memory so a captured graph
// replays it.
constexpr int kMaxBatch = 8;
template <class S>
struct MultiHop {
    HopArgs<S> a[kMaxBatch];
    int ls[kMaxBatch];
    int gx[kMaxBatch];
    long first[kMaxBatch + 1];
    int n;
};
bool multi_hop_ls(int Ls);  // Ls handled by the multi-lattice kernel
template <class S>
int launch_multi_hop(const MultiHop<S>* dev, long items, int Ls, bool dag, bool eph, bool epa,
                     bool cg, hipStream_t st);
// Whether a launch onto Vh sites of each of ndom domains (cg: with the fused update)
// takes the small-launch kernel.  hop_body's time hardly depends on the size up to 65536
// entries; the small kernel's steps up with every round of the workgroups that the CUs
// hold at once, in FP64 2 a CU (1 at Ls = 24 and 32), in FP32 and FP16 3 (2 at Ls = 32,
// and for FP16 with the update).  Microseconds of the four hops of a step, hop_body /
// small, by workgroups:
//   FP64, a second round still pays up to Ls = 12 and for single ones at Ls = 24:
//     Ls = 8  256: 68 / 36, 512: 70 / 49, 640: 71 / 62; 12  512: 65 / 47, 640: 66 / 60
//     Ls = 16 512: 63 / 52, 576: 62 / 65; 20  512: 62 / 50, 640: 62 / 64
//     Ls = 24 256: 61 / 36, 512: 62 / 59, 640: 63 / 78; 32  256: 58 / 41, 320: 59 / 63
//   FP32: 8  640: 55 / 37; 16  640: 50 / 40; 20  683: 49 / 40
//     Ls = 24 768: 50 / 40, 800: 51 / 53; 32  512: 51 / 39, 640: 50 / 58
//   FP16 without the update: 8  640: 35 / 27; 24  768: 35 / 30, 800: 33 / 40;
//     32  512: 35 / 28, 640: 35 / 41; with it 8  512: 11 / 9, 640: 12 / 15;
//     16  512: 11 / 10, 640: 11 / 15; 24  512: 11 / 9, 640: 11 / 15
// Beyond 42000 entries a CG iteration in FP64 took 137 / 142 us at 12^4 x 8 and 156 / 188
// at 12^4 x 12.
template <class S>
inline bool hop_is_small(long Vh, int Ls, int ndom, bool cg) {
    const int spb = 64 / Ls;
    const long groups = (Vh + spb - 1) / spb * ndom;
    long most = 768;
    if (sizeof(typename S::real) == 8) {
        if (Ls > 12) most = Ls <= 24 ? 512 : 256;
    } else if (Ls > 24 || (S::has_scale && cg)) {
        most = 512;
    }
    return Vh * Ls * ndom <= 42000 && groups <= most;
}
// workgroups per domain for Vh output sites on each of ndom domains; small: the
// small-launch kernel may be used
template <class S>
inline long hop_grid_x(long Vh, int Ls, int ndom, bool small, bool cg) {
    const int spb = small && hop_is_small<S>(Vh, Ls, ndom, cg) ? 64 / Ls : 256 / Ls;
    return (Vh + spb - 1) / spb;
}

// Whether an FP16 block hop onto Vh sites of each of ndom domains takes the
// matrix-core kernel (never one with the fused update, see there); inner, widest: sites
// of a block and of the largest box of a domain.  Ls = 16 fills the columns of its matrix
// instruction (with Ls = 12 in them, 24^4 in 12^4 blocks, six local steps took 6138 us
// against the general kernel's 5657).  It needs enough sites for strips of some length
// on every wave slot, and it walks whole boxes in strips and forms absent neighbours as
// zeros, where the general kernel leaves out both the corners and the neighbours: in
// small blocks most of the widened box is rim.  Hops u + y + v of a step, general /
// matrix-core us (block: part of its widened box): in favour 24^4 in 12^4 (0.32) 780 /
// 713, in 6x12x12x24 (0.34) 758 / 656, in two blocks (0.75) 514 / 434, 24^3x48 in 12^3x24
// (0.36) 1372 / 1201, in 8^3x16 (0.24) 1622 / 1517, 16x24x28x32 in 4x12x14x16 (0.23) 919 /
// 884; against 48x16^3 in 12x8^3 (0.222) 521 / 522 (a step 664 / 688), 24^4 in 24x6^3
// (0.216; a step 1118 / 1127), in 8^4 (0.20) 911 / 924, in 6^4 (0.13) 1086 / 1171, in 4^4 (0.06)
// 1553 / 2149, and with fewer sites in the blocks 16^3x32 (65536) in 8^4 364 / 416,
// 20^4 (80000) in 10^4 (0.26) 387 / 419.  A field's part of the largest box stays below
// the reach of its 32-bit offsets.
template <class S>
inline bool hop_is_rows(long Vh, long inner, long widest, int Ls, int ndom) {
    return S::has_scale && Ls == 16 && Vh * ndom >= 150000 && inner * ndom >= 90000 &&
           9 * inner > 2 * widest && widest * Ls * 48 < 0x70000000;
}
// Whether a block hop visits its sites in the order of the traversal tile: the general
// kernel onto a whole box
template <class S>
inline bool hop_follows_tile(const HopArgs<S>& a, int Ls, int ndom, bool small,
                             const HopReach* reach) {
    if (a.site_list) return false;
    if (small && hop_is_small<S>(a.g.out.Vh, Ls, ndom, a.cg_r.data != nullptr)) return false;
    return !(reach && !a.cg_r.data && hop_is_rows<S>(a.g.out.Vh, reach->inner, reach->widest, Ls, ndom));
}
constexpr int kRowWaves = 4;  // waves (strip pieces) of a workgroup
inline long row_grid_x(const Box& out, int ndom) {
    const int n = row_chunk(out, ndom);
    const long pieces = (long)out.E[1] * out.E[2] * out.E[3] / 8 * ((out.E[0] + n - 1) / n);
    return (pieces + kRowWaves - 1) / kRowWaves;
}

// out = P(in) on one box per domain (optionally |out|^2 partials).
template <class S>
struct FiveDArgs {
    CField<S> in;
    Field<S> out;
    long Vh;  // sites per domain
    FiveDProg p;
    double mf;
    double* partials;
    const int* done;
    // optional search-direction update before the program: in = src + beta in,
    // written back through xp_in (the same field as `in`); beta is
    // xp_beta[domain] when given, else xp_sc->beta
    CField<S> xp_src;
    Field<S> xp_in;
    const DevScalars* xp_sc;
    const double* xp_beta;
    // optional, with the update above: zd_z (+)= zd_alpha[domain] * (in before
    // the update); zd_z = that product when zd_first
    Field<S> zd_z;
    const double* zd_alpha;
    int zd_first;
};
template <class S>
int launch_fived(const FiveDArgs<S>& a, int Ls, int ndom, hipStream_t st);
long fived_grid_x(long Vh, int Ls);

// ---- layout conversion -------------------------------------------------
// boundary full field complex128 [Ls][Lt][Lz][Ly][Lx][4][3] <-> one parity of
// the internal whole-lattice layout.
template <class S>
int launch_pack_parity(const double2* full, Field<S> out, const int dims[4], int Ls, int par,
                       hipStream_t st);
// The same for parities par0 .. par0 + npar - 1 (fields indexed from par0), with a
// 5D program on the way: out[k] = the parity's field (data null: not stored),
// t[k] = P of it (data null: not formed).
template <class S>
int launch_pack_prog(const double2* full, const Field<S>* out, const Field<S>* t,
                     const FiveDProg& P, double mf, const int dims[4], int Ls, int par0, int npar,
                     hipStream_t st);
// full_out = P(full_in) on every site, boundary fields, arithmetic of S
template <class S>
int launch_prog_full(const double2* full_in, double2* full_out, const FiveDProg& P, double mf,
                     const int dims[4], int Ls, hipStream_t st);
template <class S>
int launch_unpack_parity(CField<S> in, double2* full, const int dims[4], int Ls, int par,
                         int zero_other, hipStream_t st);

// internal whole-lattice parity field <-> per-domain interior fields.  The
// domain grid is nb[4] blocks of extent blk[4]; domain d's origin is at
// blk * (d decomposed x-fastest).
template <class SG, class SD>
int launch_global_to_domain(CField<SG> g, Field<SD> dom, const int dims[4], const int blk[4],
                            const int nb[4], int Ls, int par, hipStream_t st);
template <class SD, class SG>
int launch_domain_to_global(CField<SD> dom, Field<SG> g, const int dims[4], const int blk[4],
                            const int nb[4], int Ls, int par, hipStream_t st);
// Even-parity domain_to_global into FP64 with the workgroup partials of
// Re<z, r> (partials[0, np)) and Re<z, q> (partials[np, 2 np)); returns np,
// or -1 on a launch error.
template <class SD>
long launch_domain_to_global_dots(CField<SD> dom, Field<F64> z, CField<F64> r, CField<F64> q,
                                  const int dims[4], const int blk[4], const int nb[4], int Ls,
                                  double* partials, hipStream_t st);

// Links for the link box of every domain (whole lattice: one domain, pad 0).
// U: boundary complex128 [4][Lt][Lz][Ly][Lx][3][3].
template <class S>
int launch_pack_links(const double2* U, typename S::elem* out, const int dims[4], const int blk[4],
                      const int nb[4], const Box& linkbox, int antiperiodic_t, hipStream_t st);

// ---- BLAS-1 and reductions ---------------------------------------------
// All vector kernels work on N = ndom*Vh*Ls elements per component; a 2D
// grid (x: chunks within a domain, y: domain) gives per-domain partial sums.
long blas_grid_x(long per_dom);

// Scalars of one solve, kept on the device.
struct DevScalars {
    double rr;       // current |r|^2 (iterated)
    double pq;       // <p, A p>
    double alpha;
    double beta;
    double zr;       // <z, r>   (flexible PCG)
    double zq;       // <z_new, q>
    double tol2;     // tol^2 |b|^2
    double bb;       // |b|^2
    int done;        // iterated residual reached tol2
    int iter;        // iterations done
    int breakdown;   // non-positive curvature or NaN
};

int launch_reduce_sum(const double* partials, int nparts, double* out, hipStream_t st);
// per-domain sums: partials [ndom][nparts] -> out[ndom]
int launch_reduce_domains(const double* partials, int ndom, int nparts, double* out,
                          hipStream_t st);

// CG scalar updates (single thread kernels)
int launch_cg_alpha(DevScalars* sc, const double* partials, int nparts, hipStream_t st,
                    int flexible = 0);
int launch_fpcg_beta(DevScalars* sc, const double* partials, int nparts, double* hist,
                     int hist_cap, hipStream_t st);
int launch_cg_beta(DevScalars* sc, const double* partials, int nparts, double* hist,
                   int hist_cap, hipStream_t st);

// FP64 whole-lattice vector kernels
int launch_sub_norm(double2* r, const double2* b, const double2* ax, long N, double* partials,
                    long nparts, hipStream_t st);
int launch_copy_norm(double2* dst, const double2* src, long N, double* partials, long nparts,
                     hipStream_t st);
int launch_dot2(const double2* z, const double2* r, const double2* q, long N, double* partials,
                long nparts, hipStream_t st);
int launch_zero(double2* y, long N, hipStream_t st);
// x += z on N whole-lattice entries (skipped when *done)
int launch_xpy(double2* x, const double2* z, long N, const int* done, hipStream_t st);
// y = a x on n complex values (any layout)
int launch_scale(double2* y, const double2* x, double a, long n, hipStream_t st);

// FP32 iterations of the mixed-precision CG
int launch_accum32(double2* x, float2* xs, long N, int Ls, hipStream_t st);

// Mixed-precision conversions (whole vectors)
template <class SI, class SO>
int launch_convert(CField<SI> in, Field<SO> out, long n_sites, hipStream_t st);

}  // namespace mspcg

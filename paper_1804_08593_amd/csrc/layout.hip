// Layout conversion kernels: boundary (lexicographic complex128) fields to the
// internal parity / domain layouts, link packing, and precision conversion.
#include "common.h"
#include "fived.h"
#include "kernels.h"

namespace mspcg {

namespace {

constexpr int kThreads = 256;

__device__ __forceinline__ void lex_coords(long lex, const int L[4], int c[4]) {
    c[0] = (int)(lex % L[0]);
    lex /= L[0];
    c[1] = (int)(lex % L[1]);
    lex /= L[1];
    c[2] = (int)(lex % L[2]);
    c[3] = (int)(lex / L[2]);
}

__device__ __forceinline__ long lex_of(const int c[4], const int L[4]) {
    return (((long)c[3] * L[2] + c[2]) * L[1] + c[1]) * L[0] + c[0];
}

struct Dims {
    int L[4];
};

// whole-lattice parity field: site cb of parity par -> lexicographic index
__device__ __forceinline__ long cb_to_lex(long cb, int par, const Dims& d) {
    Box b;
    for (int m = 0; m < 4; ++m) {
        b.E[m] = d.L[m];
        b.off[m] = 0;
    }
    b.Vh = 0;
    int c[4];
    box_coords(b, cb, par, c);
    return lex_of(c, d.L);
}

// lex index of each of the workgroup's sites (parity par, sites first, first + 1, ..)
template <int SPB>
__device__ __forceinline__ void site_lex(int* lexs, long first, long Vh, int par, const Dims& d) {
    if ((int)threadIdx.x < SPB) {
        const long cb = first + threadIdx.x;
        lexs[threadIdx.x] = cb < Vh ? (int)cb_to_lex(cb, par, d) : -1;
    }
}

// the 5D program on the LDS array, one (site, component) chain per thread
template <typename T, int LS>
__device__ __forceinline__ void prog_lds(cx<T>* lds, const FiveDProg& P, T mf) {
    constexpr int SPB = 256 / LS;
    for (int ch = (int)threadIdx.x; ch < SPB * 12; ch += (int)blockDim.x) {
        cx<T>* col = lds + ch * (LS + 1);
        cx<T> v[LS];
#pragma unroll
        for (int t = 0; t < LS; ++t) v[t] = col[t];
        apply_prog<LS, T>(P, ch % 12 < 6, mf, v);
#pragma unroll
        for (int t = 0; t < LS; ++t) col[t] = v[t];
    }
}

template <class S>
struct PackArgs {
    const double2* full;
    Field<S> out[2], t[2];  // by parity - par0; data null: not wanted
    FiveDProg p;
    double mf;
    Dims d;
    int par0;
    long V4, Vh;
};

// Boundary field -> internal parity fields, and a 5D program of them in the same
// pass (blockIdx.y: parity).  Bound by HBM: one parity with B and both outputs at
// 24^3x48x16 617 us, against 469 for the pack and 376 for the 5D kernel apart; the
// pack alone at 16^3x32x12 59 us (67 with each thread reading its own 192 bytes; 84
// with the LDS staging's loads waited for one by one).
template <class S, int LS>
__global__ __launch_bounds__(256) void pack_prog_kernel(PackArgs<S> a) {
    using T = typename S::real;
    constexpr int SPB = 256 / LS;
    __shared__ __attribute__((aligned(16))) cx<T> lds[SPB * 12 * (LS + 1)];
    __shared__ int lexs[SPB];
    const int k = blockIdx.y, sl = threadIdx.x / LS, s = threadIdx.x - sl * LS;
    const long first = (long)blockIdx.x * SPB;
    site_lex<SPB>(lexs, first, a.Vh, a.par0 + k, a.d);
    __syncthreads();
    load_boundary<T, LS>(lds, lexs, a.full, a.V4);
    __syncthreads();
    const bool active = sl < SPB && first + sl < a.Vh;
    const Field<S> out = k ? a.out[1] : a.out[0], t = k ? a.t[1] : a.t[0];
    cx<T> v[12];
    if (active && out.data) {
#pragma unroll
        for (int c = 0; c < 12; ++c) v[c] = lds[(sl * 12 + c) * (LS + 1) + s];
        store_spinor_at<S>(out, (first + sl) * LS, s, LS, v);
    }
    if (!t.data) return;
    __syncthreads();
    prog_lds<T, LS>(lds, a.p, (T)a.mf);
    __syncthreads();
    if (active) {
#pragma unroll
        for (int c = 0; c < 12; ++c) v[c] = lds[(sl * 12 + c) * (LS + 1) + s];
        store_spinor_at<S>(t, (first + sl) * LS, s, LS, v);
    }
}

// P on every site of a boundary field (blockIdx.y: parity)
template <class S, int LS>
__global__ __launch_bounds__(256) void prog_full_kernel(const double2* in, double2* out,
                                                        FiveDProg p, double mf, Dims d, long V4,
                                                        long Vh) {
    using T = typename S::real;
    constexpr int SPB = 256 / LS;
    __shared__ __attribute__((aligned(16))) cx<T> lds[SPB * 12 * (LS + 1)];
    __shared__ int lexs[SPB];
    site_lex<SPB>(lexs, (long)blockIdx.x * SPB, Vh, blockIdx.y, d);
    __syncthreads();
    load_boundary<T, LS>(lds, lexs, in, V4);
    __syncthreads();
    prog_lds<T, LS>(lds, p, (T)mf);
    __syncthreads();
    store_boundary<T, LS>(lds, lexs, out, V4, 0, (int)blockDim.x);
}

// Internal parity field -> boundary field.
template <class S, int LS>
__global__ __launch_bounds__(256) void unpack_parity_kernel(CField<S> in, double2* full, Dims d,
                                                            int par, int zero_other, long V4,
                                                            long Vh) {
    using T = typename S::real;
    constexpr int SPB = 256 / LS;
    __shared__ __attribute__((aligned(16))) cx<T> lds[SPB * 12 * (LS + 1)];
    __shared__ int lexs[SPB];
    const int sl = threadIdx.x / LS, s = threadIdx.x - sl * LS;
    const long first = (long)blockIdx.x * SPB;
    site_lex<SPB>(lexs, first, Vh, par, d);
    if (sl < SPB && first + sl < Vh) {
        cx<T> v[12];
        load_spinor_at<S, true>(in, (first + sl) * LS, s, LS, v);
#pragma unroll
        for (int c = 0; c < 12; ++c) lds[(sl * 12 + c) * (LS + 1) + s] = v[c];
    }
    __syncthreads();
    store_boundary<T, LS>(lds, lexs, full, V4, zero_other, (int)blockDim.x);
}

struct DomGrid {
    int L[4], blk[4], nb[4];
};

// domain d, interior site cb (parity par) -> global cb of the same site
__device__ __forceinline__ long dom_to_global_cb(const DomGrid& g, int d, long cb, int par) {
    Box b;
    for (int m = 0; m < 4; ++m) {
        b.E[m] = g.blk[m];
        b.off[m] = 0;
    }
    b.Vh = 0;
    int c[4];
    box_coords(b, cb, par, c);
    int dc[4];
    int r = d;
    for (int m = 0; m < 4; ++m) {
        dc[m] = r % g.nb[m];
        r /= g.nb[m];
    }
    int gcoord[4];
    for (int m = 0; m < 4; ++m) gcoord[m] = dc[m] * g.blk[m] + c[m];
    return lex_of(gcoord, g.L) >> 1;
}

template <class SG, class SD>
__global__ void global_to_domain_kernel(CField<SG> gl, Field<SD> dom, DomGrid g, int Ls, int par,
                                        long Vhb) {
    const long cb = (long)blockIdx.x * (blockDim.x / Ls) + threadIdx.x / Ls;
    const int s = threadIdx.x % Ls;
    const int d = blockIdx.y;
    if (threadIdx.x >= (blockDim.x / Ls) * Ls || cb >= Vhb) return;
    const long gcb = dom_to_global_cb(g, d, cb, par);
    cx<typename SG::real> v[12];
    load_spinor<SG>(gl, gcb * Ls + s, v);
    cx<typename SD::real> w[12];
#pragma unroll
    for (int c = 0; c < 12; ++c) w[c] = {(typename SD::real)v[c].re, (typename SD::real)v[c].im};
    store_spinor<SD>(dom, ((long)d * Vhb + cb) * Ls + s, w);
}

template <class SD, class SG>
__global__ void domain_to_global_kernel(CField<SD> dom, Field<SG> gl, DomGrid g, int Ls, int par,
                                        long Vhb) {
    const long cb = (long)blockIdx.x * (blockDim.x / Ls) + threadIdx.x / Ls;
    const int s = threadIdx.x % Ls;
    const int d = blockIdx.y;
    if (threadIdx.x >= (blockDim.x / Ls) * Ls || cb >= Vhb) return;
    const long gcb = dom_to_global_cb(g, d, cb, par);
    cx<typename SD::real> v[12];
    load_spinor<SD>(dom, ((long)d * Vhb + cb) * Ls + s, v);
    cx<typename SG::real> w[12];
#pragma unroll
    for (int c = 0; c < 12; ++c) w[c] = {(typename SG::real)v[c].re, (typename SG::real)v[c].im};
    store_spinor<SG>(gl, gcb * Ls + s, w);
}

// domain_to_global into an FP64 field z plus the workgroup partials of
// Re<z, r> and Re<z, q> (r, q: FP64 fields of the same layout as z), laid
// out [domain][workgroup] for each of the two sums, np entries apart.
template <class SD>
__global__ void domain_to_global_dots_kernel(CField<SD> dom, Field<F64> gl, CField<F64> r,
                                             CField<F64> q, DomGrid g, int Ls, long Vhb,
                                             double* partials, long np) {
    __shared__ double ra[kThreads], rb[kThreads];
    const long cb = (long)blockIdx.x * (blockDim.x / Ls) + threadIdx.x / Ls;
    const int s = threadIdx.x % Ls;
    const int d = blockIdx.y;
    double a = 0, b = 0;
    if (threadIdx.x < (blockDim.x / Ls) * Ls && cb < Vhb) {
        const long gcb = dom_to_global_cb(g, d, cb, 0);
        cx<typename SD::real> v[12];
        load_spinor<SD>(dom, ((long)d * Vhb + cb) * Ls + s, v);
        cx<double> w[12], rv[12], qv[12];
#pragma unroll
        for (int c = 0; c < 12; ++c) w[c] = {(double)v[c].re, (double)v[c].im};
        store_spinor<F64>(gl, gcb * Ls + s, w);
        load_spinor<F64>(r, gcb * Ls + s, rv);
        load_spinor<F64>(q, gcb * Ls + s, qv);
#pragma unroll
        for (int c = 0; c < 12; ++c) {
            a += w[c].re * rv[c].re + w[c].im * rv[c].im;
            b += w[c].re * qv[c].re + w[c].im * qv[c].im;
        }
    }
    // fixed-order tree over the workgroup (blockDim.x need not be a power of 2)
    const int t = threadIdx.x;
    ra[t] = a;
    rb[t] = b;
    __syncthreads();
    for (int o = kThreads / 2; o > 0; o >>= 1) {
        if (t < o && t + o < (int)blockDim.x) {
            ra[t] += ra[t + o];
            rb[t] += rb[t + o];
        }
        __syncthreads();
    }
    if (t == 0) {
        const long k = (long)d * gridDim.x + blockIdx.x;
        partials[k] = ra[0];
        partials[np + k] = rb[0];
    }
}

// One thread per (domain, parity, link-box site, direction).
template <class S>
__global__ void pack_links_kernel(const double2* U, typename S::elem* out, DomGrid g, Box lb,
                                  int antiperiodic_t, long V4) {
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    const int d = blockIdx.y;
    // consecutive threads take the 8 directions of one site (contiguous output)
    if (i >= 2 * 8 * lb.Vh) return;
    const long ps = i >> 3;
    const int dir = (int)(i & 7);
    const int par = (int)(ps / lb.Vh);
    const long cb = ps - par * lb.Vh;
    int c[4];
    box_coords(lb, cb, par, c);
    int dc[4];
    int r = d;
    for (int m = 0; m < 4; ++m) {
        dc[m] = r % g.nb[m];
        r /= g.nb[m];
    }
    int x[4];
    for (int m = 0; m < 4; ++m) {
        x[m] = dc[m] * g.blk[m] + c[m] + lb.off[m];
        x[m] = ((x[m] % g.L[m]) + g.L[m]) % g.L[m];
    }
    const int mu = dir & 3;
    const bool bwd = dir >= 4;
    double sign = 1.0;
    int y[4] = {x[0], x[1], x[2], x[3]};
    if (bwd) {
        y[mu] -= 1;
        if (y[mu] < 0) {
            y[mu] += g.L[mu];
            if (mu == 3 && antiperiodic_t) sign = -1.0;
        }
    } else if (mu == 3 && antiperiodic_t && x[3] == g.L[3] - 1) {
        sign = -1.0;
    }
    const double2* u = U + ((long)mu * V4 + lex_of(y, g.L)) * 9;
    const long obase = (long)d * (2 * 72 * lb.Vh) + ((long)par * lb.Vh + cb) * 72;
#pragma unroll
    for (int k = 0; k < 9; ++k) {
        const int row = k / 3, col = k % 3;
        double2 v;
        if (bwd) {  // (U^+)_{row,col} = conj(U_{col,row})
            const double2 t = u[col * 3 + row];
            v = make_double2(sign * t.x, -sign * t.y);
        } else {
            const double2 t = u[k];
            v = make_double2(sign * t.x, sign * t.y);
        }
        typename S::elem e;
        if constexpr (S::has_scale) {
            e = __floats2half2_rn((float)v.x, (float)v.y);
        } else {
            e.x = (typename S::real)v.x;
            e.y = (typename S::real)v.y;
        }
        out[obase + link_slot<S>(dir, k)] = e;
    }
}

template <class SI, class SO>
__global__ void convert_kernel(CField<SI> in, Field<SO> out, long n) {
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    cx<typename SI::real> v[12];
    load_spinor<SI>(in, i, v);
    cx<typename SO::real> w[12];
#pragma unroll
    for (int c = 0; c < 12; ++c) w[c] = {(typename SO::real)v[c].re, (typename SO::real)v[c].im};
    store_spinor<SO>(out, i, w);
}

inline unsigned nblocks(long n, int t) { return (unsigned)((n + t - 1) / t); }

int last_error() { return hipGetLastError() == hipSuccess ? 0 : -2; }

}  // namespace

template <class S>
int launch_pack_prog(const double2* full, const Field<S>* out, const Field<S>* t,
                     const FiveDProg& P, double mf, const int dims[4], int Ls, int par0, int npar,
                     hipStream_t st) {
    PackArgs<S> a = {};
    a.full = full;
    for (int k = 0; k < npar; ++k) {
        if (out) a.out[k] = out[k];
        if (t) a.t[k] = t[k];
    }
    a.p = P;
    a.mf = mf;
    a.d = Dims{{dims[0], dims[1], dims[2], dims[3]}};
    a.par0 = par0;
    a.V4 = (long)dims[0] * dims[1] * dims[2] * dims[3];
    a.Vh = a.V4 / 2;
    switch (Ls) {
#define MSPCG_CASE(L)                                                                             \
    case L:                                                                                       \
        hipLaunchKernelGGL((pack_prog_kernel<S, L>), dim3(nblocks(a.Vh, 256 / L), npar), dim3(256), \
                           0, st, a);                                                             \
        break;
        MSPCG_LS_LIST(MSPCG_CASE)
#undef MSPCG_CASE
        default: return -1;
    }
    return last_error();
}

template <class S>
int launch_pack_parity(const double2* full, Field<S> out, const int dims[4], int Ls, int par,
                       hipStream_t st) {
    return launch_pack_prog<S>(full, &out, nullptr, FiveDProg{}, 0.0, dims, Ls, par, 1, st);
}

template <class S>
int launch_prog_full(const double2* full_in, double2* full_out, const FiveDProg& P, double mf,
                     const int dims[4], int Ls, hipStream_t st) {
    Dims d{{dims[0], dims[1], dims[2], dims[3]}};
    const long V4 = (long)dims[0] * dims[1] * dims[2] * dims[3], Vh = V4 / 2;
    switch (Ls) {
#define MSPCG_CASE(L)                                                                            \
    case L:                                                                                      \
        hipLaunchKernelGGL((prog_full_kernel<S, L>), dim3(nblocks(Vh, 256 / L), 2), dim3(256), 0, \
                           st, full_in, full_out, P, mf, d, V4, Vh);                             \
        break;
        MSPCG_LS_LIST(MSPCG_CASE)
#undef MSPCG_CASE
        default: return -1;
    }
    return last_error();
}

template <class S>
int launch_unpack_parity(CField<S> in, double2* full, const int dims[4], int Ls, int par,
                         int zero_other, hipStream_t st) {
    Dims d{{dims[0], dims[1], dims[2], dims[3]}};
    const long V4 = (long)dims[0] * dims[1] * dims[2] * dims[3];
    const long Vh = V4 / 2;
    switch (Ls) {
#define MSPCG_CASE(L)                                                                             \
    case L:                                                                                       \
        hipLaunchKernelGGL((unpack_parity_kernel<S, L>), dim3(nblocks(Vh, 256 / L)), dim3(256), 0, \
                           st, in, full, d, par, zero_other, V4, Vh);                             \
        break;
        MSPCG_LS_LIST(MSPCG_CASE)
#undef MSPCG_CASE
        default: return -1;
    }
    return last_error();
}

static DomGrid make_grid(const int dims[4], const int blk[4], const int nb[4]) {
    DomGrid g;
    for (int m = 0; m < 4; ++m) {
        g.L[m] = dims[m];
        g.blk[m] = blk[m];
        g.nb[m] = nb[m];
    }
    return g;
}

template <class SG, class SD>
int launch_global_to_domain(CField<SG> gl, Field<SD> dom, const int dims[4], const int blk[4],
                            const int nb[4], int Ls, int par, hipStream_t st) {
    const DomGrid g = make_grid(dims, blk, nb);
    const long Vhb = (long)blk[0] * blk[1] * blk[2] * blk[3] / 2;
    const int spb = kThreads / Ls;
    const int ndom = nb[0] * nb[1] * nb[2] * nb[3];
    hipLaunchKernelGGL((global_to_domain_kernel<SG, SD>), dim3(nblocks(Vhb, spb), ndom),
                       dim3(spb * Ls), 0, st, gl, dom, g, Ls, par, Vhb);
    return last_error();
}

template <class SD, class SG>
int launch_domain_to_global(CField<SD> dom, Field<SG> gl, const int dims[4], const int blk[4],
                            const int nb[4], int Ls, int par, hipStream_t st) {
    const DomGrid g = make_grid(dims, blk, nb);
    const long Vhb = (long)blk[0] * blk[1] * blk[2] * blk[3] / 2;
    const int spb = kThreads / Ls;
    const int ndom = nb[0] * nb[1] * nb[2] * nb[3];
    hipLaunchKernelGGL((domain_to_global_kernel<SD, SG>), dim3(nblocks(Vhb, spb), ndom),
                       dim3(spb * Ls), 0, st, dom, gl, g, Ls, par, Vhb);
    return last_error();
}

template <class SD>
long launch_domain_to_global_dots(CField<SD> dom, Field<F64> gl, CField<F64> r, CField<F64> q,
                                  const int dims[4], const int blk[4], const int nb[4], int Ls,
                                  double* partials, hipStream_t st) {
    const DomGrid g = make_grid(dims, blk, nb);
    const long Vhb = (long)blk[0] * blk[1] * blk[2] * blk[3] / 2;
    const int spb = kThreads / Ls;
    const int ndom = nb[0] * nb[1] * nb[2] * nb[3];
    const long gx = nblocks(Vhb, spb);
    const long np = gx * ndom;
    hipLaunchKernelGGL((domain_to_global_dots_kernel<SD>), dim3((unsigned)gx, ndom),
                       dim3(spb * Ls), 0, st, dom, gl, r, q, g, Ls, Vhb, partials, np);
    return last_error() ? -1 : np;
}

template <class S>
int launch_pack_links(const double2* U, typename S::elem* out, const int dims[4], const int blk[4],
                      const int nb[4], const Box& lb, int antiperiodic_t, hipStream_t st) {
    const DomGrid g = make_grid(dims, blk, nb);
    const long V4 = (long)dims[0] * dims[1] * dims[2] * dims[3];
    const int ndom = nb[0] * nb[1] * nb[2] * nb[3];
    hipLaunchKernelGGL(pack_links_kernel<S>, dim3(nblocks(2 * 8 * lb.Vh, kThreads), ndom),
                       dim3(kThreads), 0, st, U, out, g, lb, antiperiodic_t, V4);
    return last_error();
}

template <class SI, class SO>
int launch_convert(CField<SI> in, Field<SO> out, long n, hipStream_t st) {
    hipLaunchKernelGGL((convert_kernel<SI, SO>), dim3(nblocks(n, kThreads)), dim3(kThreads), 0, st,
                       in, out, n);
    return last_error();
}

#define MSPCG_INST0(S)                                                                             \
    template int launch_pack_prog<S>(const double2*, const Field<S>*, const Field<S>*,            \
                                     const FiveDProg&, double, const int*, int, int, int,         \
                                     hipStream_t);                                                 \
    template int launch_prog_full<S>(const double2*, double2*, const FiveDProg&, double,          \
                                     const int*, int, hipStream_t);                                \
    template int launch_pack_parity<S>(const double2*, Field<S>, const int*, int, int,            \
                                       hipStream_t);                                               \
    template int launch_unpack_parity<S>(CField<S>, double2*, const int*, int, int, int,          \
                                         hipStream_t);
MSPCG_INST0(F64)
MSPCG_INST0(F32)
#define MSPCG_INST1(S)                                                                             \
    template int launch_pack_links<S>(const double2*, typename S::elem*, const int*, const int*,  \
                                      const int*, const Box&, int, hipStream_t);
MSPCG_INST1(F64)
MSPCG_INST1(F32)
MSPCG_INST1(F16)
#define MSPCG_INST_DOTS(S)                                                                         \
    template long launch_domain_to_global_dots<S>(CField<S>, Field<F64>, CField<F64>, CField<F64>, \
                                                  const int*, const int*, const int*, int,         \
                                                  double*, hipStream_t);
MSPCG_INST_DOTS(F64)
MSPCG_INST_DOTS(F32)
MSPCG_INST_DOTS(F16)
#define MSPCG_INST2(A, B)                                                                          \
    template int launch_global_to_domain<A, B>(CField<A>, Field<B>, const int*, const int*,       \
                                               const int*, int, int, hipStream_t);                 \
    template int launch_domain_to_global<B, A>(CField<B>, Field<A>, const int*, const int*,       \
                                               const int*, int, int, hipStream_t);                 \
    template int launch_convert<A, B>(CField<A>, Field<B>, long, hipStream_t);                     \
    template int launch_convert<B, A>(CField<B>, Field<A>, long, hipStream_t);
MSPCG_INST2(F64, F16)
MSPCG_INST2(F64, F32)
MSPCG_INST2(F32, F16)
template int launch_global_to_domain<F64, F64>(CField<F64>, Field<F64>, const int*, const int*,
                                               const int*, int, int, hipStream_t);
template int launch_domain_to_global<F64, F64>(CField<F64>, Field<F64>, const int*, const int*,
                                               const int*, int, int, hipStream_t);
template int launch_global_to_domain<F32, F32>(CField<F32>, Field<F32>, const int*, const int*,
                                               const int*, int, int, hipStream_t);
template int launch_domain_to_global<F32, F32>(CField<F32>, Field<F32>, const int*, const int*,
                                               const int*, int, int, hipStream_t);

}  // namespace mspcg

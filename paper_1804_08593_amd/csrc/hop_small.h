// The Wilson hop for launches too small to fill the GPU: the eight directions
// of a site run in the eight waves of a workgroup.
//
// hop_body gives each (site, s) to one thread, which visits the directions one
// after another; when every workgroup of a launch is resident at once, its time
// is that thread's chain of eight dependent memory latencies.  Here wave D of a
// workgroup loads, projects and multiplies direction D only, for 64 / Ls sites,
// and the half spinors are summed over the directions from LDS in hop_body's
// order (wave c sums colour-spin component c of the upper and of the lower
// two spins), so the result is the same to the last bit; partial sums are
// grouped by the smaller workgroups.
//
#pragma once
#include "hop_impl.h"

namespace mspcg {

constexpr int kSmallThreads = 512;

// component c of entry (base + s)
template <class S>
__device__ __forceinline__ long comp_index(long base, int s, int ls, int c) {
    constexpr int V = Chunk<S>::V, K = Chunk<S>::K;
    if constexpr (S::has_scale) return (base * K + (long)(c % 3) * ls + s) * V + c / 3;
    return (base * K + (long)(c / V) * ls + s) * V + c % V;
}
template <class S>
__device__ __forceinline__ cx<typename S::real> load_comp(CField<S> f, long base, int s, int ls,
                                                          int c) {
    cx<typename S::real> v = elem_cx<S>(f.data[comp_index<S>(base, s, ls, c)]);
    if constexpr (S::has_scale) {
        const float k = f.scale[base + s];
        v.re *= k;
        v.im *= k;
    }
    return v;
}
template <class S>
__device__ __forceinline__ void store_comp(Field<S> f, long base, int s, int ls, int c,
                                           cx<typename S::real> v) {
    typename S::elem e;
    e.x = v.re;
    e.y = v.im;
    f.data[comp_index<S>(base, s, ls, c)] = e;
}

template <class S, int LS, bool DAG, bool CG>
__global__ __launch_bounds__(kSmallThreads) void hop_small_kernel(HopArgs<S> a) {
    using T = typename S::real;
    using E = typename S::elem;
    constexpr int SPB = 64 / LS;  // sites of a workgroup
    // half spinors [direction][6][64] (and FP16 scales), then the 5D exchange
    // arrays [12][64] of the hop result and of aux in the same place
    __shared__ __attribute__((aligned(16))) cx<T> lds[8 * 6 * 64];
    __shared__ float lk[S::has_scale ? 8 * 64 : 1];
    if (a.done && *a.done) return;
    int bx, d;
    logical_block(a.xcd_remap, bx, d);
    const HopGeom& g = a.g;
    const int e = (int)(threadIdx.x & 63);
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int sl = e / LS, s = e - sl * LS;
    const long t_lin = (long)bx * SPB + sl;
    const bool active = sl < SPB && t_lin < (a.site_list ? a.n_list : g.out.Vh);
    long cb = t_lin;
    int gc[4] = {0, 0, 0, 0};
    if (active) {
        int oc[4];
        if (a.site_list) cb = a.site_list[t_lin];
        box_coords(g.out, cb, g.out_par, oc);
#pragma unroll
        for (int m = 0; m < 4; ++m) gc[m] = oc[m] + g.out.off[m];
    }
    const long obase = ((long)d * g.out.Vh + cb) * LS;
    // aux components c and 6 + c of wave c < 6, loaded ahead of the products
    cx<T> xu = {0, 0}, xd = {0, 0};
    if (a.has_aux && wv < 6 && active) {
        int ac[4];
        bool in = true;
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            ac[m] = gc[m] - g.aux.off[m];
            in = in && ac[m] >= 0 && ac[m] < g.aux.E[m];
        }
        if (in) {
            const long ab = ((long)d * g.aux.Vh + box_cb(g.aux, ac)) * LS;
            xu = load_comp<S>(a.aux, ab, s, LS, wv);
            xd = load_comp<S>(a.aux, ab, s, LS, 6 + wv);
        }
    }

    // direction wv: w = U (psi_up + sig e psi_dn) of the neighbour
    constexpr int SF = DAG ? 1 : -1;
    constexpr int SB = -SF;
    sfor<8>([&](auto di) {
        constexpr int D = decltype(di)::value;
        constexpr int MU = D / 2;
        constexpr bool FWD = (D % 2) == 0;
        if (wv != D) return;
        cx<T> w[6];
#pragma unroll
        for (int c = 0; c < 6; ++c) w[c] = {0, 0};
        float k = 0.f;
        if (active) {
            const InPos ip = in_position(g, gc);
            long n = 0;
            if (neighbour<MU, FWD ? 1 : 0>(g, ip, n)) {
                RawSpinor<S> raw;
                load_raw_at<S>(a.in, ((long)d * g.in.Vh + n) * LS, s, LS, raw);
                int lc[4];
#pragma unroll
                for (int m = 0; m < 4; ++m) lc[m] = gc[m] - g.link.off[m];
                const E* gl = a.links + (long)d * a.link_dom_stride +
                              ((long)g.out_par * g.link.Vh + box_cb(g.link, lc)) * 72;
                cx<T> u[9];
#pragma unroll
                for (int q = 0; q < 9; ++q) u[q] = load_link<S>(gl + link_slot<S>(FWD ? MU : 4 + MU, q));
                cx<T> p[12], h[6];
                decode_raw<S>(raw, p, false);
                project<MU, FWD ? SF : SB, false>(p, h, (T)1);
#pragma unroll
                for (int sp = 0; sp < 2; ++sp)
#pragma unroll
                    for (int i = 0; i < 3; ++i) {
                        cx<T> t = cmul(u[i * 3 + 0], h[sp * 3 + 0]);
                        cfma(t, u[i * 3 + 1], h[sp * 3 + 1]);
                        cfma(t, u[i * 3 + 2], h[sp * 3 + 2]);
                        w[sp * 3 + i] = t;
                    }
                if constexpr (S::has_scale) k = raw.sc;
            }
        }
#pragma unroll
        for (int c = 0; c < 6; ++c) lds[(D * 6 + c) * 64 + e] = w[c];
        if constexpr (S::has_scale) lk[D * 64 + e] = k;
    });
    // What the fused update reads of components c and 6 + c of wave c < 6, all before
    // the first store: a load behind a store waits for a latency of its own.  Ahead of
    // the products its registers came on top of theirs (FP64 at Ls = 6 .. 16 130-132
    // VGPRs against 104-116, one workgroup a CU instead of two: Ls = 8, 512 workgroups
    // 15.9 us against 12.5; 256 workgroups 9.9 and 10.3).  LATE: behind the 5D programs,
    // where their vectors along s would cost a workgroup of a CU again (FP64 Ls = 16, 512
    // workgroups 17.3 -> 13.3 us; FP32 Ls = 20, 640 workgroups 14.8 -> 11.0).
    constexpr bool LATE = sizeof(T) == 8 ? LS == 16 || LS == 20 : LS == 20 || LS == 24;
    cx<T> cr[2], cp[2], cxv[2];
    T al = 0;
    auto operands = [&]() {
        if constexpr (CG && !S::has_scale) {
            al = (T)(a.cg_alpha ? a.cg_alpha[d] : a.cg_sc->alpha);
            if (wv < 6 && active) {
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int q = wv + 6 * h;
                    cr[h] = load_comp<S>(cfield(a.cg_r), obase, s, LS, q);
                    cp[h] = cxv[h] = {0, 0};
                    if (a.cg_x.data) {
                        cp[h] = load_comp<S>(a.cg_p, obase, s, LS, q);
                        if (!a.cg_first) cxv[h] = load_comp<S>(cfield(a.cg_x), obase, s, LS, q);
                    }
                }
            }
        }
    };
    if constexpr (!LATE) operands();
    __syncthreads();

    // wave c = 3 sp + colour < 6: the sums of components c and 6 + c (reconstruct)
    const int c = wv;
    cx<T> ru = {0, 0}, rd = {0, 0};
    if (c < 6) {
        const int sp = c >= 3, pc = sp ? c - 3 : c + 3;
        sfor<8>([&](auto di) {
            constexpr int D = decltype(di)::value;
            constexpr int MU = D / 2;
            const T sg = (T)((D % 2) == 0 ? SF : SB);
            const T k = S::has_scale ? (T)lk[D * 64 + e] : (T)1;
            const cx<T> w = lds[(D * 6 + c) * 64 + e];
            ru.re = fmadd(k, w.re, ru.re);
            ru.im = fmadd(k, w.im, ru.im);
            if constexpr (MU == 0) {
                const cx<T> q = lds[(D * 6 + pc) * 64 + e];
                rd.re = fmadd(k, -sg * q.im, rd.re);
                rd.im = fmadd(k, sg * q.re, rd.im);
            } else if constexpr (MU == 1) {
                const cx<T> q = lds[(D * 6 + pc) * 64 + e];
                const T f = sp ? -sg : sg;
                rd.re = fmadd(k, f * q.re, rd.re);
                rd.im = fmadd(k, f * q.im, rd.im);
            } else if constexpr (MU == 2) {
                const T f = sp ? -sg : sg;
                rd.re = fmadd(k, -f * w.im, rd.re);
                rd.im = fmadd(k, f * w.re, rd.im);
            } else {
                rd.re = fmadd(k, sg * w.re, rd.re);
                rd.im = fmadd(k, sg * w.im, rd.im);
            }
        });
    }

    // 5D programs through LDS: component-major arrays [12][64], the hop result
    // first, aux behind it
    const T mf = (T)a.mf;
    cx<T>* lh = lds;
    cx<T>* lx = lds + 12 * 64;
    const bool hp = !a.ph.identity, xp = a.has_aux && !a.pa.identity;
    if (hp || xp) {
        __syncthreads();  // the half spinors are read
        if (c < 6) {
            if (hp) lh[c * 64 + e] = ru, lh[(6 + c) * 64 + e] = rd;
            if (xp) lx[c * 64 + e] = xu, lx[(6 + c) * 64 + e] = xd;
        }
        __syncthreads();
        const int nch = (hp ? SPB * 12 : 0) + (xp ? SPB * 12 : 0);
        for (int t = (int)threadIdx.x; t < nch; t += kSmallThreads) {
            const bool first = hp && t < SPB * 12;
            const int q = hp && !first ? t - SPB * 12 : t;
            cx<T>* col = (first ? lh : lx) + (q / SPB) * 64 + (q % SPB) * LS;
            cx<T> v[LS];
#pragma unroll
            for (int k = 0; k < LS; ++k) v[k] = col[k];
            apply_prog<LS, T>(first ? a.ph : a.pa, q / SPB < 6, mf, v);
#pragma unroll
            for (int k = 0; k < LS; ++k) col[k] = v[k];
        }
        __syncthreads();
        if (c < 6) {
            if (hp) ru = lh[c * 64 + e], rd = lh[(6 + c) * 64 + e];
            if (xp) xu = lx[c * 64 + e], xd = lx[(6 + c) * 64 + e];
        }
    }
    if constexpr (LATE) operands();
    if (a.ph.identity) {
        ru.re *= (T)a.ph.scale[0], ru.im *= (T)a.ph.scale[0];
        rd.re *= (T)a.ph.scale[1], rd.im *= (T)a.ph.scale[1];
    }
    if (a.has_aux) {
        const T su = a.pa.identity ? (T)a.pa.scale[0] : (T)1, sd = a.pa.identity ? (T)a.pa.scale[1] : (T)1;
        ru.re += su * xu.re, ru.im += su * xu.im;
        rd.re += sd * xd.re, rd.im += sd * xd.im;
    }

    double n2 = 0;
    if constexpr (S::has_scale) {
        // an FP16 entry is stored with one scale: wave 0 gathers the components
        __syncthreads();
        if (c < 6) lh[c * 64 + e] = ru, lh[(6 + c) * 64 + e] = rd;
        __syncthreads();
        if (wv == 0 && active) {
            cx<T> res[12], v[12];
#pragma unroll
            for (int q = 0; q < 12; ++q) res[q] = lh[q * 64 + e];
            T t2 = 0;
            if (!CG || a.cg_keep_out) store_spinor_at<S>(a.out, obase, s, LS, res);
            if constexpr (CG) {
                const T al = (T)(a.cg_alpha ? a.cg_alpha[d] : a.cg_sc->alpha);
                load_spinor_at<S>(cfield(a.cg_r), obase, s, LS, v);
#pragma unroll
                for (int q = 0; q < 12; ++q) {
                    v[q].re -= al * res[q].re;
                    v[q].im -= al * res[q].im;
                    t2 = fmadd(v[q].re, v[q].re, t2);
                    t2 = fmadd(v[q].im, v[q].im, t2);
                }
                store_spinor_at<S>(a.cg_r, obase, s, LS, v);
                if (a.cg_x.data) {
                    cx<T> pv[12];
                    load_spinor_at<S>(a.cg_p, obase, s, LS, pv);
                    if (!a.cg_first) load_spinor_at<S>(cfield(a.cg_x), obase, s, LS, v);
#pragma unroll
                    for (int q = 0; q < 12; ++q) {
                        v[q].re = a.cg_first ? al * pv[q].re : v[q].re + al * pv[q].re;
                        v[q].im = a.cg_first ? al * pv[q].im : v[q].im + al * pv[q].im;
                    }
                    store_spinor_at<S>(a.cg_x, obase, s, LS, v);
                }
            } else {
#pragma unroll
                for (int q = 0; q < 12; ++q) {
                    t2 = fmadd(res[q].re, res[q].re, t2);
                    t2 = fmadd(res[q].im, res[q].im, t2);
                }
            }
            n2 = (double)t2;
        }
    } else if (c < 6 && active) {
        if (!CG && a.bout) {
            const long lex = 2 * cb + (gc[0] & 1);
            double2* o = a.bout + ((long)s * a.V4 + lex) * 12 + c;
            o[0] = make_double2(ru.re, ru.im);
            o[6] = make_double2(rd.re, rd.im);
            if (a.zero_other) {
                o += lex & 1 ? -12 : 12;
                o[0] = o[6] = make_double2(0.0, 0.0);
            }
        } else if (!CG || a.cg_keep_out) {
            store_comp<S>(a.out, obase, s, LS, c, ru);
            store_comp<S>(a.out, obase, s, LS, 6 + c, rd);
        }
        T t2 = 0;
        auto square = [&](cx<T> v) {
            t2 = fmadd(v.re, v.re, t2);
            t2 = fmadd(v.im, v.im, t2);
        };
        if constexpr (CG) {
            // r -= alpha out, x += alpha p
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int q = c + 6 * h;
                const cx<T> o = h ? rd : ru;
                cx<T> v = cr[h];
                v.re -= al * o.re;
                v.im -= al * o.im;
                square(v);
                store_comp<S>(a.cg_r, obase, s, LS, q, v);
                if (a.cg_x.data) {
                    cx<T> x = {al * cp[h].re, al * cp[h].im};
                    if (!a.cg_first) {
                        x = cxv[h];
                        x.re += al * cp[h].re;
                        x.im += al * cp[h].im;
                    }
                    store_comp<S>(a.cg_x, obase, s, LS, q, x);
                }
            }
        } else {
            square(ru);
            square(rd);
        }
        n2 = (double)t2;
    }
    if (CG || a.partials) block_sum_store<S, LS>(n2, a.partials + (long)d * gridDim.x + bx);
}

template <class S, int LS>
void launch_small_ls(const HopArgs<S>& a, int ndom, bool dag, hipStream_t st) {
    constexpr int SPB = 64 / LS;
    const long nout = a.site_list ? a.n_list : a.g.out.Vh;
    const dim3 grid((unsigned)((nout + SPB - 1) / SPB), (unsigned)ndom), block(kSmallThreads);
    if (a.cg_r.data)
        hipLaunchKernelGGL((hop_small_kernel<S, LS, true, true>), grid, block, 0, st, a);
    else if (dag)
        hipLaunchKernelGGL((hop_small_kernel<S, LS, true, false>), grid, block, 0, st, a);
    else
        hipLaunchKernelGGL((hop_small_kernel<S, LS, false, false>), grid, block, 0, st, a);
}

template <class S>
int launch_hop_small(const HopArgs<S>& a, int Ls, int ndom, bool dag, hipStream_t st) {
    switch (Ls) {
#define MSPCG_CASE(L) \
    case L: launch_small_ls<S, L>(a, ndom, dag, st); break;
        MSPCG_LS_LIST(MSPCG_CASE)
#undef MSPCG_CASE
        default: return -1;
    }
    return 0;
}

}  // namespace mspcg

// FP16-storage Wilson hop on the matrix cores (gfx950): a wave walks a strip of
// output sites along x, the fifth dimension along the 16 lanes of a row.
//
// For each direction the wave forms w = U (psi_up + sig e psi_dn), the six
// complex rows that the projector (1 + sig g_mu) keeps, as one
// v_mfma_f32_16x16x32_f16 with the s slices as the 16 columns:
//   B  column s, K chunk j: the four spins (re, im) of colour j of the
//      neighbour, which is the 16-byte chunk j of the FP16 layout.  Lane
//      (j, s) loads its chunk and it is the operand as it stands; the fourth
//      K chunk is zero.
//   A  row 4 i + r: colour i of (Re w0, Im w0, Re w1, Im w1)[r]; K chunk j
//      holds U_ij times the spin projector: U_ij on the row's own spin, and
//      U_ij times +-1 or +-i on its partner spin.  A lane reads one link
//      entry and places its halves (or their negatives) by byte permutes
//      with lane-constant selectors.
//   D  lane (i, s) holds both kept rows of colour i, so the reconstruction of
//      the lower two spins stays within the lane, and the result has the
//      lane layout of the inputs.
// FP16 products are exact and summed in FP32; the neighbour's FP32 scale
// multiplies the sum as it is added to the accumulators, as in hop_body.
//
// A strip is 2 x 2 x 2 sites in (y, z, t) (every box extent is even): of its 8
// corners 4 are outputs at each x and the other 4 inputs.  The inputs inside
// the strip stay in registers for the three x at which they are used, so an
// output costs 4 neighbour loads instead of 8; the address unit takes 16 to 20
// cycles for a vector load whatever its width, so scales and links are loaded
// for several neighbours at once.
// Everything that belongs to the site (indices, bounds) is the same in the
// whole wave and runs on the scalar unit; a dropped hop reads through a buffer
// descriptor of length zero, which returns zeros without touching memory.
//
// 24^3 x 48 x 16 in 16 blocks, hops u / y / v of the block operator: 317 / 450 / 330 us
// (general kernel 373 / 524 / 400).  v is bound by what passes between L2 and memory, 6.2
// TB/s; u (3.4 TB/s) by its vector instructions, issued 71% of the time (233 an output,
// 96 of them the scaled sums); y (4.8 TB/s, 65%) lies between.  More waves than 3 a SIMD
// need registers that spill (u 393 us at 4).  The hop with the fused update stays with
// the general kernel: here it took 306 us, 489 with the update of x (there 326 on
// average), and left the 5D kernel behind it less in cache (277 against 250 us).
// The 5D programs move values along s with DPP row shifts instead of LDS.
//
#pragma once
#include "hop_impl.h"

namespace mspcg {

namespace rows {

constexpr int LS = 16;  // the columns of a matrix instruction

typedef _Float16 row_h8 __attribute__((ext_vector_type(8)));
typedef float row_f4 __attribute__((ext_vector_type(4)));

// Buffer descriptor of `bytes` at p (the same in the whole wave): reads past
// the end return zero, writes past the end are dropped.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t row_rsrc(const void* p, int bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, bytes, 0x00027000);
}

// y[i] += c * (y[i] of the lane that the DPP control selects; 0 beyond the row's
// end), as one instruction each.  Written out because the compiler keeps the
// lane move and the multiply-add apart.  s_nop 1: the two wait states between
// a vector write and its read through DPP.
#define MSPCG_ROW_FMAC(NAME, CTRL)                                                                \
    template <int N>                                                                              \
    __device__ __forceinline__ void NAME(float (&y)[4], float c) {                                \
        asm("s_nop 1\n\t"                                                                         \
            "v_fmac_f32_dpp %0, %0, %4 " CTRL ":%5 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"   \
            "v_fmac_f32_dpp %1, %1, %4 " CTRL ":%5 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"   \
            "v_fmac_f32_dpp %2, %2, %4 " CTRL ":%5 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"   \
            "v_fmac_f32_dpp %3, %3, %4 " CTRL ":%5 row_mask:0xf bank_mask:0xf bound_ctrl:1"       \
            : "+v"(y[0]), "+v"(y[1]), "+v"(y[2]), "+v"(y[3])                                      \
            : "v"(c), "n"(N));                                                                    \
    }
MSPCG_ROW_FMAC(row_fmac_shr, "row_shr")
MSPCG_ROW_FMAC(row_fmac_shl, "row_shl")
MSPCG_ROW_FMAC(row_fmac_ror, "row_ror")
MSPCG_ROW_FMAC(row_fmac_bcast, "row_newbcast")
#undef MSPCG_ROW_FMAC

// Lane constants of a 5D program's bidiagonal step: what a lane adds of its
// neighbour below (b) and above (a), the corner closing the s direction.
struct RowBidi {
    float b, a;
    __device__ __forceinline__ void set(const RowProg& P, int s) {
        b = s == 0 ? P.corner : P.a;
        a = s == LS - 1 ? P.corner : P.a;
    }
};
// ... and of its inverse step: powers of q and e_s for the neighbour below, above
struct RowInv {
    float q1, q2, q4, q8, eb, ea;
};

// v_s += f v_{s-1} (below) or f v_{s+1} (above)
template <bool BELOW>
__device__ __forceinline__ void row_bidi(float (&x)[4], const RowBidi& k) {
    row_fmac_ror<BELOW ? 1 : 15>(x, BELOW ? k.b : k.a);
}

// (1 - q K)^-1 along the row: t_s = sum_{k <= s} q^(s-k) x_k by a scan, then
// y_s = t_s + e_s t_end with e_s = -mf q^(s+1) / (1 + mf q^Ls);
// mirrored for the other direction.
template <bool BELOW>
__device__ __forceinline__ void row_inv(float (&x)[4], const RowInv& k) {
    if constexpr (BELOW) {
        row_fmac_shr<1>(x, k.q1);
        row_fmac_shr<2>(x, k.q2);
        row_fmac_shr<4>(x, k.q4);
        row_fmac_shr<8>(x, k.q8);
        row_fmac_bcast<LS - 1>(x, k.eb);
    } else {
        row_fmac_shl<1>(x, k.q1);
        row_fmac_shl<2>(x, k.q2);
        row_fmac_shl<4>(x, k.q4);
        row_fmac_shl<8>(x, k.q8);
        row_fmac_bcast<0>(x, k.ea);
    }
}

// The 8 reals of one colour at one (site, s): the upper two spins (re, im) and
// the lower two.
struct RowHalf {
    float u[4], d[4];
};

// One 5D program on them.  K takes psi_{s-1} on the upper chirality, K^+ (the
// dagger hop's programs) on the lower one.
template <bool DAG, bool INV>
__device__ __forceinline__ void row_prog(const RowProg& P, const RowBidi& kb, const RowInv& ki,
                                         RowHalf& v) {
    if (DAG && P.bidi) {
        row_bidi<false>(v.u, kb);
        row_bidi<true>(v.d, kb);
    }
    if constexpr (INV) {
        row_inv<!DAG>(v.u, ki);
        row_inv<DAG>(v.d, ki);
    }
    if (!DAG && P.bidi) {
        row_bidi<true>(v.u, kb);
        row_bidi<false>(v.d, kb);
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        v.u[c] *= P.su;
        v.d[c] *= P.sd;
    }
}

// The launch arguments, read anew through the scalar cache: an opaque copy of
// the pointer keeps a loop from holding every argument in scalar registers
// (which spilled them to vector registers).
template <class T>
__device__ __forceinline__ const T& row_args(const T* p) {
    auto q = (const __attribute__((address_space(4))) T*)p;
    asm volatile("" : "+s"(q));
    return *(const T*)q;
}

// byte selectors of v_perm over (-u, u): halves re, im, -re, -im
constexpr unsigned row_sel(unsigned lo, unsigned hi) { return (hi << 16) | lo; }
constexpr unsigned kRe = 0x0100, kIm = 0x0302, kNRe = 0x0504, kNIm = 0x0706, kZero = 0x0c0c0c0cu;

// A domain's part of a field.  A domain's bytes stay below 4 GB, so a site is
// a 32-bit scalar offset.
struct RowField {
    const char* data;
    const float* scale;
    unsigned sites;
    template <class F>
    __device__ __forceinline__ void set(const F& f, int d, long vh) {
        data = reinterpret_cast<const char*>(f.data) + (long)d * vh * (LS * 48);
        scale = f.scale + (long)d * vh * LS;
        sites = (unsigned)vh;
    }
};

// One entry as loaded: a chunk of the spinor and its scale.
struct RowSite {
    nt_u4 d;
    float k;
};

// the chunk at `site` (zeros when not ok)
__device__ __forceinline__ nt_u4 row_data(const RowField& f, int site, bool ok, int lane_off) {
    return __builtin_amdgcn_raw_buffer_load_b128(row_rsrc(f.data, ok ? (int)(f.sites * (LS * 48)) : 0),
                                                 lane_off, ok ? site * (LS * 48) : 0, 0);
}

// rows 0 .. 3 of a value, each spread over all four rows
__device__ __forceinline__ void row_spread(float v, float (&r)[4]) {
    float a = v, b, a2, b2;
    asm("v_mov_b32 %1, %0\n\t"
        "s_nop 1\n\t"
        "v_permlane32_swap_b32 %0, %1\n\t"
        "s_nop 1\n\t"
        "v_mov_b32 %2, %0\n\t"
        "v_mov_b32 %3, %1\n\t"
        "s_nop 1\n\t"
        "v_permlane16_swap_b32 %0, %2\n\t"
        "v_permlane16_swap_b32 %1, %3\n\t"
        "s_nop 1"
        : "+v"(a), "=&v"(b), "=&v"(a2), "=&v"(b2));
    r[0] = a;
    r[1] = a2;
    r[2] = b;
    r[3] = b2;
}

// the entry at `site` (zeros when not ok); AUX: cache policy (2: read once)
template <int AUX>
__device__ __forceinline__ RowSite row_load(const RowField& f, int site, bool ok, int lane_off,
                                            int sc_off) {
    RowSite r;
    site = ok ? site : 0;
    r.d = __builtin_amdgcn_raw_buffer_load_b128(row_rsrc(f.data, ok ? (int)(f.sites * (LS * 48)) : 0),
                                                lane_off, site * (LS * 48), AUX);
    r.k = __builtin_bit_cast(
        float, __builtin_amdgcn_raw_buffer_load_b32(row_rsrc(f.scale, ok ? (int)(f.sites * (LS * 4)) : 0),
                                                    sc_off, site * (LS * 4), AUX));
    return r;
}

__device__ __forceinline__ void row_decode(const RowSite& r, RowHalf& v) {
    const cx<float> a = h2f(r.d.x, r.k), b = h2f(r.d.y, r.k);
    const cx<float> c = h2f(r.d.z, r.k), e = h2f(r.d.w, r.k);
    v.u[0] = a.re, v.u[1] = a.im, v.u[2] = b.re, v.u[3] = b.im;
    v.d[0] = c.re, v.d[1] = c.im, v.d[2] = e.re, v.d[3] = e.im;
}

// an entry to be stored: max-scaled halves and the scale
__device__ __forceinline__ RowSite row_encode(const RowHalf& v) {
    // scale: max |real| over the entry's 24 reals, 8 in each of three rows
    float m = 0.f;
#pragma unroll
    for (int c = 0; c < 4; ++c)
        asm("v_max3_f32 %0, |%1|, |%2|, %0" : "+v"(m) : "v"(v.u[c]), "v"(v.d[c]));
    // over the four rows; written out because the compiler folds the maximum of
    // the two results of a lane swap into one of them
    float t1;
    asm("v_mov_b32 %1, %0\n\t"
        "s_nop 1\n\t"
        "v_permlane32_swap_b32 %0, %1\n\t"
        "s_nop 1\n\t"
        "v_max_f32 %0, %0, %1\n\t"
        "v_mov_b32 %1, %0\n\t"
        "s_nop 1\n\t"
        "v_permlane16_swap_b32 %0, %1\n\t"
        "s_nop 1\n\t"
        "v_max_f32 %0, %0, %1"
        : "+v"(m), "=&v"(t1));
    const float inv = m > 0.f ? 1.0f / m : 0.f;
    RowSite r;
    r.k = m;
    r.d = nt_u4{f2h(v.u[0] * inv, v.u[1] * inv), f2h(v.u[2] * inv, v.u[3] * inv),
                f2h(v.d[0] * inv, v.d[1] * inv), f2h(v.d[2] * inv, v.d[3] * inv)};
    return r;
}

// (nothing when not ok); AUX: cache policy
template <int AUX>
__device__ __forceinline__ void row_store(const RowField& f, int site, bool ok, int lane_off, int sc_off,
                                          const RowSite& r) {
    const unsigned n = __builtin_amdgcn_readfirstlane(ok ? f.sites : 0u);
    site = __builtin_amdgcn_readfirstlane(ok ? site : 0);
    __builtin_amdgcn_raw_buffer_store_b128(r.d, row_rsrc(f.data, (int)(n * (LS * 48))), lane_off,
                                           site * (LS * 48), AUX);
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, r.k),
                                          row_rsrc(f.scale, (int)(n * (LS * 4))), sc_off,
                                          site * (LS * 4), AUX);
}

// One workgroup's share of a hop launch: strip pieces [bx*kRowWaves,
// (bx+1)*kRowWaves) of domain d, one per wave.  A piece is `chunk` steps of x of
// one strip; the pieces of a strip follow each other, so that the slices of inputs
// that two of them load are found in L2.
// INV: the hop's program holds an inverse step, and there is neither aux nor
// partials; else no inverse step.
template <bool DAG, bool INV>
__device__ __forceinline__ void row_body(const RowArgs* ap, int bx, int d, int gx) {
    const int lane = (int)(threadIdx.x & 63), grp = lane >> 4, s = lane & 15;
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    bx = __builtin_amdgcn_readfirstlane(bx);
    d = __builtin_amdgcn_readfirstlane(d);
    constexpr int SB = LS * 48;           // bytes of a site
    constexpr int OUT = (int)0xfffffff0;  // beyond every descriptor used here
    // this lane's chunk (colour grp of slice s), its scale, its link entry
    const int lane_off = grp < 3 ? (grp * LS + s) * 16 : OUT;
    const int sc_ld = s * 4;
    constexpr int NONE = 0x03000000;  // a site index whose scale lies beyond every field
    const int row = s >> 2, sp = (s >> 1) & 1, ci = s & 1;  // A row: colour, spin, re/im
    // link entry (colour row, grp) of direction 0, as the byte address of the
    // lane that loads it; lanes outside the 3 x 3 select zeros
    const bool used = grp < 3 && row < 3;
    const int link_at = used ? (row * 3 + grp) * 4 : 0;
    // selectors: the entry on spin sp = 0, 1, and times -i
    const unsigned one = ci ? row_sel(kIm, kRe) : row_sel(kRe, kNIm);
    const unsigned mi = ci ? row_sel(kNRe, kIm) : row_sel(kIm, kRe);  // times -i
    const unsigned s0 = used && !sp ? one : kZero, s1 = used && sp ? one : kZero;
    const unsigned m0 = used && !sp ? mi : kZero, m1 = used && sp ? mi : kZero;

    // the piece: its x range, and the rows (site index at x = 0 of the row's box) of
    // the sites around the strip, one per lane: the 8 corners in the input box, the
    // y, z, t neighbours outside the strip of corner c at 8 + 3 c + {0, 1, 2}, and
    // the corners in the output, link and aux box at 32, 40, 48.  valid: lanes whose
    // row exists.
    int xlo, xhi, rows;
    unsigned valid, valid_aux = 0;
    int in_x, in_E, link_x, aux_x = 0, aux_E = 0, out_E;  // box x = output x + *_x (periodic: in_E < 0)
    // sites that matter: distance `left` remains for x; bit m of far (3 + m): corner
    // bit m clear (set) is a site further from the block; block range in x
    int left = 1 << 20, bx0 = 0, bx1 = 1 << 20;
    unsigned far = 0;
    RowBidi kh, ka;
    RowInv ki;
    RowField in, out, aux;
    const char* linkp;
    RowProg ph, pa;
    {
        const RowArgs& a = row_args(ap);
        const HopGeom& g = a.g;
        const unsigned n1 = (unsigned)g.out.E[1] >> 1, n2 = (unsigned)g.out.E[2] >> 1,
                       n3 = (unsigned)g.out.E[3] >> 1;
        const unsigned it = (unsigned)bx * kRowWaves + (unsigned)wv;
        const unsigned pieces = (unsigned)((g.out.E[0] + a.chunk - 1) / a.chunk);
        unsigned q = it / pieces;
        const unsigned piece = it - q * pieces;
        const unsigned r = q / n1;
        int ob[4];  // domain coordinates of corner 0
        ob[1] = 2 * (int)(q - r * n1) + g.out.off[1];
        ob[3] = 2 * (int)(r / n2) + g.out.off[3];
        ob[2] = 2 * (int)(r % n2) + g.out.off[2];
        // corners of even coordinate sum are outputs at x = phase (mod 2); pieces
        // begin there
        const int phase =
            (g.out_par + g.out.off[0] + g.out.off[1] + g.out.off[2] + g.out.off[3]) & 1;
        out_E = g.out.E[0];
        xlo = (int)piece * a.chunk - phase;
        xhi = ((int)piece + 1) * a.chunk >= out_E ? out_E : xlo + a.chunk;
        if (q >= n1 * n2 * n3) xhi = xlo;  // waves beyond the last piece
        if (a.reach >= 0) {
            left = a.reach;
            if (a.blk[0]) {
                bx0 = -g.out.off[0];
                bx1 = a.blk[0] - g.out.off[0];
            }
#pragma unroll
            for (int m = 1; m < 4; ++m) {
                const int lo = ob[m];
                if (!a.blk[m]) continue;
                left -= lo + 1 < 0 ? -(lo + 1) : (lo >= a.blk[m] ? lo - a.blk[m] + 1 : 0);
                if (lo < 0) far |= 1u << (m - 1);
                if (lo + 1 >= a.blk[m]) far |= 8u << (m - 1);
            }
            if (left < 0) xhi = xlo;
            while (xlo + 2 <= bx0 - left) xlo += 2;
            xhi = xhi < bx1 + left ? xhi : bx1 + left;
        }
        {
            // this lane's row
            const bool nb = lane >= 8 && lane < 32;
            const int c = nb ? (lane - 8) / 3 : lane & 7, dim = nb ? (lane - 8) % 3 : 3;
            const int kind = lane < 32 ? 0 : (lane - 24) >> 3;  // input, output, link, aux (4: none)
            int y[4];
            int E[4], of[4];
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                E[m] = kind == 0 ? g.in.E[m] : kind == 1 ? g.out.E[m] : kind == 2 ? g.link.E[m] : g.aux.E[m];
                of[m] = kind == 0   ? g.in.off[m]
                        : kind == 1 ? g.out.off[m]
                        : kind == 2 ? g.link.off[m]
                                    : g.aux.off[m];
            }
            bool ok = lane < 56;
#pragma unroll
            for (int m = 1; m < 4; ++m) {
                const int bit = (c >> (m - 1)) & 1;
                y[m] = ob[m] - of[m] + (dim == m - 1 ? (bit ? 2 : -1) : bit);
                if (kind == 0 && ((g.periodic >> m) & 1))
                    y[m] = y[m] < 0 ? y[m] + E[m] : (y[m] >= E[m] ? y[m] - E[m] : y[m]);
                ok = ok && (unsigned)y[m] < (unsigned)E[m];
            }
            rows = ok ? ((y[3] * E[2] + y[2]) * E[1] + y[1]) * (E[0] >> 1) : NONE;
            const unsigned long b = __ballot(ok);
            valid = (unsigned)b;
            if constexpr (!INV) valid_aux = a.has_aux ? (unsigned)(b >> 48) & 0xffu : 0u;
        }
        in.set(a.in, d, g.in.Vh);
        in_x = g.out.off[0] - g.in.off[0];
        in_E = g.periodic & 1 ? -g.in.E[0] : g.in.E[0];
        out.set(a.out, d, g.out.Vh);
        linkp = reinterpret_cast<const char*>(a.links + (long)d * a.link_dom_stride +
                                              (long)g.out_par * g.link.Vh * 72);
        link_x = g.out.off[0] - g.link.off[0];
        ph = a.rh;
        kh.set(a.rh, s);
        if constexpr (INV) {
            // e_s: cinv q^(s+1) from below, cinv q^(LS-s) from above
            const float q1 = a.rh.q, q2 = q1 * q1, q4 = q2 * q2, q8 = q4 * q4;
            auto power = [&](int n) {
                float f = n & 1 ? q1 : 1.f;
                f *= n & 2 ? q2 : 1.f;
                f *= n & 4 ? q4 : 1.f;
                f *= n & 8 ? q8 : 1.f;
                return n & 16 ? f * q8 * q8 : f;
            };
            ki = {q1, q2, q4, q8, a.rh.cinv * power(s + 1), a.rh.cinv * power(LS - s)};
            // kept in vector registers, as the lane moves need them
            asm volatile("" : "+v"(ki.q1), "+v"(ki.q2), "+v"(ki.q4), "+v"(ki.q8));
        } else {
            aux.set(a.aux, d, g.aux.Vh);
            aux_x = g.out.off[0] - g.aux.off[0];
            aux_E = g.aux.E[0];
            pa = a.ra;
            ka.set(a.ra, s);
        }
    }
    double n2 = 0;

    // x part of the input sites at output coordinate x, and the rows that exist there
    struct XPos {
        int xs;
        unsigned ok;
    };
    auto at = [&](int x) {
        const int E = in_E < 0 ? -in_E : in_E;
        int xi = x + in_x;
        if (in_E < 0) xi = xi < 0 ? xi + E : (xi >= E ? xi - E : xi);
        return XPos{xi >> 1, (unsigned)xi < (unsigned)E ? valid : 0u};
    };
    auto fetch = [&](int row, const XPos& p) {
        return row_load<0>(in, __builtin_amdgcn_readlane(rows, row) + p.xs, (p.ok >> row) & 1,
                               lane_off, sc_ld);
    };
    // what is loaded ahead of an output: the y, z, t neighbours outside the strip,
    // their scales in rows 0, 1, 2 of `k` with the scale of the input that is
    // refilled next in row 3 (one load instead of four: a vector memory instruction
    // costs the address unit the same whatever its width), and the links, forward
    // and backward entry in lane 9 mu + entry
    struct Ahead {
        nt_u4 h[3];
        float k;
        unsigned uf, ub;
    };
    auto issue = [&](auto cc, int x, const XPos& p, int refill, const XPos& pr, Ahead& b) {
        constexpr int C = decltype(cc)::value;
        const int lx = (x < 0 ? 0 : (x < out_E ? x : out_E - 1)) + link_x;
        const unsigned n = (unsigned)(__builtin_amdgcn_readlane(rows, 40 + C) + (lx >> 1));
        typedef unsigned u2 __attribute__((ext_vector_type(2)));
        const u2 l = __builtin_amdgcn_raw_buffer_load_b64(
            row_rsrc(linkp + (unsigned long)n * 288, 288), lane * 8, 0, 0);
        b.uf = l.x;
        b.ub = l.y;
        const int site = __builtin_amdgcn_ds_bpermute(
                             grp == 3 ? refill * 4 : (8 + 3 * C + grp) * 4, rows) +
                         (grp == 3 ? (pr.ok ? pr.xs : NONE) : (p.ok ? p.xs : NONE));
        b.k = __builtin_bit_cast(
            float, __builtin_amdgcn_raw_buffer_load_b32(
                       row_rsrc(in.scale, (int)(in.sites * (LS * 4))),
                       (int)((unsigned)site * (LS * 4u) + s * 4u), 0, 0));
#pragma unroll
        for (int i = 0; i < 3; ++i)
            b.h[i] = row_data(in, __builtin_amdgcn_readlane(rows, 8 + 3 * C + i) + p.xs,
                                  (p.ok >> (8 + 3 * C + i)) & 1, lane_off);
    };
    // what an output reads at its own site.  Issued before the loads for the next
    // output, so that the wait for them leaves those in flight.
    struct Own {
        RowSite ya;
    };
    auto issue_own = [&](auto cc, int x, bool want, Own& o) {
        constexpr int C = decltype(cc)::value;
        // aux lives on its own box; sites outside it contribute zero
        if constexpr (!INV)
            o.ya = row_load<2>(
                aux, __builtin_amdgcn_readlane(rows, 48 + C) + ((x + aux_x) >> 1),
                want && ((valid_aux >> C) & 1) && (unsigned)(x + aux_x) < (unsigned)aux_E,
                lane_off, sc_ld);
    };
    // the output at corner C and x; hk: the scales of b.h; xm, xp: the inputs at
    // x - 1 and x + 1, own: those at x
    // want: whether it matters.  Its memory operations are issued either way
    // (nothing moves when it does not): with the same number of them on both paths
    // the wait for a load does not take in the stores issued after it.
    auto output = [&](auto cc, int x, bool want, const Own& o, const Ahead& b,
                      const float (&hk)[4], const RowSite (&xm)[4], const RowSite (&own)[4],
                      const RowSite (&xp)[4]) {
        constexpr int C = decltype(cc)::value;
        using std::integral_constant;
        RowSite so{nt_u4{0, 0, 0, 0}, 0.f};
        if (want) {
            RowHalf v;
#pragma unroll
            for (int c = 0; c < 4; ++c) v.u[c] = v.d[c] = 0.f;
            // this lane's entry of the eight links, by direction slot
            unsigned ul[8];
            sfor<8>([&](auto di) {
                constexpr int D = decltype(di)::value;
                ul[D] = (unsigned)__builtin_amdgcn_ds_bpermute(link_at + (D & 3) * 36,
                                                               (int)(D < 4 ? b.uf : b.ub));
            });
            // the eight hops in the order in which their loads were issued: 0 x -, 1..3
            // the y, z, t neighbours inside the strip, 4 x +, 5..7 those outside
            auto product = [&](auto ic) {
                constexpr int I = decltype(ic)::value, MU = I & 3;
                constexpr int bit = MU == 0 ? 1 : (C >> (MU > 0 ? MU - 1 : 0)) & 1;
                constexpr bool FWD = I < 4 ? !bit : bit;
                constexpr int SIG = FWD == DAG ? 1 : -1;  // forward 1 - g, backward 1 + g; dagger swaps
                const nt_u4& n = I == 0   ? xm[C >> 1].d
                                 : I == 1 ? own[(C ^ 1) >> 1].d
                                 : I == 2 ? own[(C ^ 2) >> 1].d
                                 : I == 3 ? own[(C ^ 4) >> 1].d
                                 : I == 4 ? xp[C >> 1].d
                                          : b.h[I >= 5 ? I - 5 : 0];
                const unsigned ud = ul[FWD ? MU : 4 + MU], un = ud ^ 0x80008000u;
                const unsigned hi = SIG > 0 ? un : ud, lo = SIG > 0 ? ud : un;
                // the partner spins 2 and 3, sig e_mu: x -i of spin 1, 0; y +1 of spin 1,
                // -1 of spin 0; z -i of spin 0, +i of spin 1; t +1 of spin 0, 1
                const unsigned a2 = MU == 0   ? __builtin_amdgcn_perm(hi, lo, m1)
                                    : MU == 1 ? __builtin_amdgcn_perm(hi, lo, s1)
                                    : MU == 2 ? __builtin_amdgcn_perm(hi, lo, m0)
                                              : __builtin_amdgcn_perm(hi, lo, s0);
                const unsigned a3 = MU == 0   ? __builtin_amdgcn_perm(hi, lo, m0)
                                    : MU == 1 ? __builtin_amdgcn_perm(lo, hi, s0)
                                    : MU == 2 ? __builtin_amdgcn_perm(lo, hi, m1)
                                              : __builtin_amdgcn_perm(hi, lo, s1);
                const nt_u4 A{__builtin_amdgcn_perm(un, ud, s0), __builtin_amdgcn_perm(un, ud, s1), a2, a3};
                return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(row_h8, A),
                                                              __builtin_bit_cast(row_h8, n),
                                                              row_f4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
            };
            auto collect = [&](auto ic, const row_f4& w) {
                constexpr int I = decltype(ic)::value, MU = I & 3;
                constexpr int bit = MU == 0 ? 1 : (C >> (MU > 0 ? MU - 1 : 0)) & 1;
                constexpr bool FWD = I < 4 ? !bit : bit;
                constexpr int SIG = FWD == DAG ? 1 : -1;
                const float q = I == 0   ? xm[C >> 1].k
                                : I == 1 ? own[(C ^ 1) >> 1].k
                                : I == 2 ? own[(C ^ 2) >> 1].k
                                : I == 3 ? own[(C ^ 4) >> 1].k
                                : I == 4 ? xp[C >> 1].k
                                         : hk[I >= 5 ? I - 5 : 0];
                const float sq = SIG > 0 ? q : -q;
#pragma unroll
                for (int c = 0; c < 4; ++c) v.u[c] = fmadd(q, w[c], v.u[c]);
                // lower spins: sig e_mu^+ w (see reconstruct)
                constexpr int src[4][4] = {{3, 2, 1, 0}, {2, 3, 0, 1}, {1, 0, 3, 2}, {0, 1, 2, 3}};
                constexpr int sgn[4][4] = {{-1, 1, -1, 1}, {1, 1, -1, -1}, {-1, 1, 1, -1}, {1, 1, 1, 1}};
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    v.d[c] = fmadd(sgn[MU][c] > 0 ? sq : -sq, w[src[MU][c]], v.d[c]);
            };
            // a product runs on the matrix core while the one before it is collected
            row_f4 w[2];
            w[0] = product(integral_constant<int, 0>{});
            sfor<7>([&](auto ii) {
                constexpr int I = decltype(ii)::value;
                w[(I + 1) & 1] = product(integral_constant<int, I + 1>{});
                __builtin_amdgcn_sched_barrier(0);
                collect(integral_constant<int, I>{}, w[I & 1]);
                __builtin_amdgcn_sched_barrier(0);
            });
            collect(integral_constant<int, 7>{}, w[1]);

            row_prog<DAG, INV>(ph, kh, ki, v);
            if constexpr (!INV) {
                RowHalf y;
                row_decode(o.ya, y);
                row_prog<DAG, false>(pa, ka, ki, y);
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    v.u[c] += y.u[c];
                    v.d[c] += y.d[c];
                }
            }
            so = row_encode(v);
            if constexpr (!INV) {
                float t2 = 0;
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    t2 = fmadd(v.u[c], v.u[c], t2);
                    t2 = fmadd(v.d[c], v.d[c], t2);
                }
                n2 += (double)t2;
            }
        }
        const int oat = __builtin_amdgcn_readlane(rows, 32 + C) + (x >> 1);
        row_store<2>(out, oat, want, lane_off, sc_ld, so);
    };

    if (xlo < xhi) {
        // A step takes the outputs at x (even corners), then those at x + 1 (odd).
        // The next output's loads are issued before an output is formed; an input's
        // register is refilled with the one three slices on as soon as its last
        // output is done.
        RowSite p0[4], p1[4], p2[4];  // inputs at x - 1, x, x + 1
        Ahead b0, b1;
        constexpr std::integral_constant<int, 0> c0{};
        constexpr std::integral_constant<int, 1> c1{};
        constexpr std::integral_constant<int, 2> c2{};
        constexpr std::integral_constant<int, 3> c3{};
        constexpr std::integral_constant<int, 4> c4{};
        constexpr std::integral_constant<int, 5> c5{};
        constexpr std::integral_constant<int, 6> c6{};
        constexpr std::integral_constant<int, 7> c7{};
        int x = xlo;
        XPos h = at(x), n = at(x - 1);
        p0[0] = fetch(0, n), p0[1] = fetch(3, n), p0[2] = fetch(5, n), p0[3] = fetch(6, n);
        p1[0] = fetch(1, h), p1[1] = fetch(2, h), p1[2] = fetch(4, h), p1[3] = fetch(7, h);
        n = at(x + 1);
        p2[0] = fetch(0, n), p2[1] = fetch(3, n), p2[2] = fetch(5, n), p2[3] = fetch(6, n);
        issue(c0, x, h, 6, n, b0);
        // the corners that matter at x (none outside the box)
        auto wanted = [&](int x) -> unsigned {
            const int dx = x < bx0 ? bx0 - x : (x >= bx1 ? x - bx1 + 1 : 0), rest = left - dx;
            if ((unsigned)x >= (unsigned)out_E || rest < 0) return 0u;
            if (rest >= 3) return 0xffu;
            unsigned w = 0;
#pragma unroll
            for (int c = 0; c < 8; ++c)
                if (__builtin_popcount(far & ((7 & ~c) | c << 3)) <= rest) w |= 1u << c;
            return w;
        };
        // filled: the input refilled in the step before, whose scale came with b
        auto step = [&](auto cc, int x, unsigned want, const Ahead& b, RowSite& filled, auto next,
                        int xn, const XPos& pn, Ahead& bn, RowSite (&xm)[4],
                        const RowSite (&own)[4], const RowSite (&xp)[4], int refill,
                        const XPos& pr) {
            constexpr int C = decltype(cc)::value;
            Own o;
            issue_own(cc, x, (want >> C) & 1, o);
            __builtin_amdgcn_sched_barrier(0);
            issue(next, xn, pn, refill, pr, bn);
            __builtin_amdgcn_sched_barrier(0);
            float hk[4];
            row_spread(b.k, hk);
            filled.k = hk[3];
            output(cc, x, (want >> C) & 1, o, b, hk, xm, own, xp);
            xm[C >> 1].d = row_data(in, __builtin_amdgcn_readlane(rows, refill) + pr.xs,
                                        (pr.ok >> refill) & 1, lane_off);
            __builtin_amdgcn_sched_barrier(0);
        };
#pragma unroll 1
        for (; x < xhi; x += 2) {
            const unsigned we = wanted(x), wo = wanted(x + 1);
            const XPos q0 = at(x), q1 = at(x + 1), q2 = at(x + 2), q3 = at(x + 3);
            step(c0, x, we, b0, p2[3], c3, x, q0, b1, p0, p1, p2, 1, q2);
            step(c3, x, we, b1, p0[0], c5, x, q0, b0, p0, p1, p2, 2, q2);
            step(c5, x, we, b0, p0[1], c6, x, q0, b1, p0, p1, p2, 4, q2);
            step(c6, x, we, b1, p0[2], c1, x + 1, q1, b0, p0, p1, p2, 7, q2);
            step(c1, x + 1, wo, b0, p0[3], c2, x + 1, q1, b1, p1, p2, p0, 0, q3);
            step(c2, x + 1, wo, b1, p1[0], c4, x + 1, q1, b0, p1, p2, p0, 3, q3);
            step(c4, x + 1, wo, b0, p1[1], c7, x + 1, q1, b1, p1, p2, p0, 5, q3);
            step(c7, x + 1, wo, b1, p1[2], c0, x + 2, q2, b0, p1, p2, p0, 6, q3);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const nt_u4 td = p0[i].d;
                const float tk = p0[i].k;
                p0[i].d = p2[i].d, p0[i].k = p2[i].k;
                p2[i].d = p1[i].d, p2[i].k = p1[i].k;
                p1[i].d = td, p1[i].k = tk;
            }
        }
    }
    if constexpr (!INV) {
        const RowArgs& a = row_args(ap);
        if (a.partials) block_sum_store<F16, LS>(n2, a.partials + (long)d * gx + bx);
    }
}

}  // namespace rows

}  // namespace mspcg

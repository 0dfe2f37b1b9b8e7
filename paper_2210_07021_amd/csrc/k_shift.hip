// Lemmas 2 and 4 (M2M, L2L) on the FP64 matrix cores.
//
// Both passes go level by level, and most levels hold too few boxes to fill
// the chip, so what counts is how long one wave takes for its translations.
// With a lane (or four) per box that is the whole 4 p^2-flop serial chain
// (19-25 us a level at p = 38, whatever the level's size; 7.4 us here, and 57
// against 41 us for the one level of 143,000 boxes).  Here a wave takes
// 16 children of the level at once: the two Taylor shifts of the factorised
// translation (expand.hpp) are products with the binomial matrix, the same
// for every pair, and v_mfma_f64_4x4x4 (four 4 x 4 blocks, 74 TFLOP/s measured
// against 65 for FMAs and 48 for the 16 x 16 x 4 form) works on all 16 columns
// with a quarter of the coefficients per lane.
//
// Layout.  Lane: column (child) lane & 15, coefficient index l = 4 r + (lane
// >> 4) in register r.  That is the B operand's layout with r as the k step,
// and a 4 x 4 x 4 result has the same layout (row lane >> 4), so the output
// tiles of the first shift are the input tiles of the second.
//
// Shift by b:  v_n = sum_l C(l, n) b^(l-n) z_l, tile t of n from tiles r >= t
// of l.  b^(l-n) = b^(4(r-t)) b^k b^-i with k, i the places in the tiles: the
// lane factors b^k and b^-i are applied before and after, and b^(4(r-t)) by
// Horner steps over r (one multiply of the running tile per step).  Nothing
// over- or underflows for any b (below 1e-60 it is taken as 1e-60, which
// changes nothing at double precision: the terms it scales are absent there).
// The transposed shift by a (second factor) is the same with t >= r.  At deep
// levels one of the two parameters is tiny (Lemma 2: b ~ 4^-level, Lemma 4:
// a): from 1e-6 down only the tiles t and t +- 1 can matter (C(64, 5) b^5 <
// 1e-22), and below 1e-19 the shift is the identity.
#include "common.hpp"
#include "expand.hpp"

namespace sfmm {

namespace {
constexpr int kTiles = kMaxOrder / 4 + 1;               // tiles of 4 over l = 0 .. kMaxOrder
constexpr int kPairs = kTiles * (kTiles + 1) / 2;       // (lower, higher) tile pairs
constexpr double kTinyShift = 1e-60, kBandShift = 1e-6, kNoShift = 1e-19;

// A operands, [pair][k][i] (lane: i = lane & 3, k = lane >> 4): up, tile row
// n = 4 lo + i, l = 4 hi + k: C(l, n); down, tile row l = 4 hi + i, n = 4 lo
// + k: C(l - 1, n - 1) (none for l or n = 0).  C(67, 33) < 2^64.
struct ShiftTab {
    double up[kPairs * 16], down[kPairs * 16], inv[4 * kTiles];
};
constexpr ShiftTab make_shift_tab() {
    ShiftTab t{};
    unsigned long long c[4 * kTiles][4 * kTiles] = {};
    for (int l = 0; l < 4 * kTiles; ++l) {
        c[l][0] = 1;
        for (int n = 1; n <= l; ++n) c[l][n] = c[l - 1][n - 1] + (n < l ? c[l - 1][n] : 0);
    }
    for (int hi = 0; hi < kTiles; ++hi)
        for (int lo = 0; lo <= hi; ++lo)
            for (int k = 0; k < 4; ++k)
                for (int i = 0; i < 4; ++i) {
                    const int at = (hi * (hi + 1) / 2 + lo) * 16 + 4 * k + i;
                    const int lu = 4 * hi + k, nu = 4 * lo + i;
                    t.up[at] = nu <= lu ? (double)c[lu][nu] : 0.0;
                    const int ld = 4 * hi + i, nd = 4 * lo + k;
                    t.down[at] = nd >= 1 && nd <= ld ? (double)c[ld - 1][nd - 1] : 0.0;
                }
    for (int l = 0; l < 4 * kTiles; ++l) t.inv[l] = l ? 1.0 / l : 0.0;
    return t;
}
__device__ const ShiftTab kShiftTab = make_shift_tab();

// a pointer into the tables that stays a global one
using TabPtr = const double __attribute__((address_space(1)))*;

__device__ __forceinline__ double mfma4(double a, double b, double c) {
    return __builtin_amdgcn_mfma_f64_4x4x4f64(a, b, c, 0, 0, 0);
}

// x^k for k = 0 .. 3 (k = lane >> 4)
__device__ __forceinline__ double pow_k(double x, int k) {
    const double x2 = x * x;
    return (k & 2 ? x2 : 1.0) * (k & 1 ? x : 1.0);
}
__device__ __forceinline__ cplx pow_k(cplx x, int k) {
    const cplx x2 = cmul(x, x);
    const cplx hi = k & 2 ? x2 : cplx{1.0, 0.0};
    return k & 1 ? cmul(hi, x) : hi;
}

// v_t = sum_{r = t}^{t + W - 1} s4^(r - t) A(t, r) z_r; tab: the lane's first
// entry of the up table.  The operands of the next r are loaded while those
// of this one are used (the barriers keep the compiler from sinking the loads
// to their uses, which leaves each one's latency bare).
template <int NT, int W>
__device__ __forceinline__ void shift_up(TabPtr tab, double s4, const double (&zr)[NT], const double (&zi)[NT],
                                         double (&vr)[NT], double (&vi)[NT]) {
    double a[2][W];
#pragma unroll
    for (int d = 0; d < W; ++d) a[(NT - 1) & 1][d] = tab[((NT - 1) * NT / 2 + (NT - 1 - d)) * 16];
#pragma unroll
    for (int r = NT - 1; r >= 0; --r) {
        if (r > 0) {
#pragma unroll
            for (int d = 0; d < W && d <= r - 1; ++d) a[(r - 1) & 1][d] = tab[((r - 1) * r / 2 + (r - 1 - d)) * 16];
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int d = 0; d < W && d <= r; ++d) {
            const int t = r - d;
            const bool first = r == (t + W - 1 < NT - 1 ? t + W - 1 : NT - 1);
            vr[t] = mfma4(a[r & 1][d], zr[r], first ? 0.0 : vr[t] * s4);
            vi[t] = mfma4(a[r & 1][d], zi[r], first ? 0.0 : vi[t] * s4);
        }
        __builtin_amdgcn_sched_barrier(0);
    }
}

// v_t = sum_{r = t - W + 1}^{t} s4^(t - r) A(t, r) z_r
template <int NT, int W>
__device__ __forceinline__ void shift_down(TabPtr tab, double s4, const double (&zr)[NT], const double (&zi)[NT],
                                           double (&vr)[NT], double (&vi)[NT]) {
    double a[2][W];
#pragma unroll
    for (int d = 0; d < W && d < NT; ++d) a[0][d] = tab[(d * (d + 1) / 2) * 16];
#pragma unroll
    for (int r = 0; r < NT; ++r) {
        if (r + 1 < NT) {
#pragma unroll
            for (int d = 0; d < W && r + 1 + d < NT; ++d)
                a[(r + 1) & 1][d] = tab[((r + 1 + d) * (r + 2 + d) / 2 + r + 1) * 16];
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int d = 0; d < W && r + d < NT; ++d) {
            const int t = r + d;
            const bool first = r == (t - W + 1 > 0 ? t - W + 1 : 0);
            vr[t] = mfma4(a[r & 1][d], zr[r], first ? 0.0 : vr[t] * s4);
            vi[t] = mfma4(a[r & 1][d], zi[r], first ? 0.0 : vi[t] * s4);
        }
        __builtin_amdgcn_sched_barrier(0);
    }
}

__device__ __forceinline__ bool any_lane(bool v) { return __ballot(v) != 0; }

// One translation per column.  in: the source record of the lane's column.
// On return (o_re, o_im)[r] is the translated A_l, l = 4 r + kq, for l = 1 ..
// P, and u0 (lanes kq = 0) the series part of C'.
template <int P>
__device__ __forceinline__ void translate_cols(const double* __restrict__ in, const TransGeom& G, int kq,
                                               double* o_re, double* o_im, double* u0) {
    constexpr int NT = P / 4 + 1;
    const int lane = threadIdx.x & 63, ti = (lane >> 4) * 4 + (lane & 3);
    // the lane's entries of the tables, as plain pointers (each load of a
    // constant place of a named array costs three scalar instructions)
    TabPtr up = (TabPtr)kShiftTab.up + ti, down = (TabPtr)kShiftTab.down + ti, inv = (TabPtr)kShiftTab.inv + kq;
    asm("" : "+v"(up), "+v"(down), "+v"(inv));
    double zr[NT], zi[NT], vr[NT], vi[NT];
    const double b = fmax(G.b, kTinyShift), a = fmax(G.a, kTinyShift);
    // input: b^k ph1^l A_l
    {
        cplx w = pow_k(G.ph1, kq);
        const cplx p2 = cmul(G.ph1, G.ph1), p4 = cmul(p2, p2);
        const double bk = pow_k(b, kq);
#pragma unroll
        for (int r = 0; r < NT; ++r) {
            const int l = 4 * r + kq;
            const double2 x = reinterpret_cast<const double2*>(in)[l < P ? l : P];
            const bool live = l >= 1 && l <= P;
            const cplx v = cmul(w, cplx{x.x * bk, x.y * bk});
            zr[r] = live ? v.re : 0.0;
            zi[r] = live ? v.im : 0.0;
            w = cmul(w, p4);
        }
    }
    const double b2 = b * b, a2 = a * a;
    if (any_lane(b > kBandShift)) {
        shift_up<NT, NT>(up, b2 * b2, zr, zi, vr, vi);
    } else if (any_lane(b > kNoShift)) {
        shift_up<NT, (NT < 2 ? NT : 2)>(up, b2 * b2, zr, zi, vr, vi);
    } else {
#pragma unroll
        for (int r = 0; r < NT; ++r) {
            vr[r] = zr[r];
            vi[r] = zi[r];
        }
    }
    // the diagonal g^n with the lane factors b^-i (first shift) and a^-k
    // (second); entry 0 only feeds C'
    const double ibk = 1.0 / pow_k(b, kq);
    *u0 = vr[0] * ibk;
    {
        const double g2 = G.g * G.g, g4 = g2 * g2;
        const double f0 = ibk / pow_k(a, kq);
        double gn = pow_k(G.g, kq);
#pragma unroll
        for (int r = 0; r < NT; ++r) {
            zr[r] = vr[r] * f0 * gn;
            zi[r] = vi[r] * f0 * gn;
            gn *= g4;
        }
    }
    if (any_lane(a > kBandShift)) {
        shift_down<NT, NT>(down, a2 * a2, zr, zi, vr, vi);
    } else if (any_lane(a > kNoShift)) {
        shift_down<NT, (NT < 2 ? NT : 2)>(down, a2 * a2, zr, zi, vr, vi);
    } else {
#pragma unroll
        for (int r = 0; r < NT; ++r) {
            vr[r] = zr[r];
            vi[r] = zi[r];
        }
    }
    // output: ph2^l (a^i v - (Q / l) a^l)
    {
        cplx w = pow_k(G.ph2, kq);
        const cplx p2 = cmul(G.ph2, G.ph2), p4 = cmul(p2, p2);
        const double ak = pow_k(a, kq), Q = in[1];
        double an = ak;
#pragma unroll
        for (int r = 0; r < NT; ++r) {
            const double re = fma(-Q * inv[4 * r], an, vr[r] * ak);
            const cplx v = cmul(w, cplx{re, vi[r] * ak});
            o_re[r] = v.re;
            o_im[r] = v.im;
            w = cmul(w, p4);
            an *= a2 * a2;
        }
    }
}

template <int CTRL>
__device__ __forceinline__ double dpp_quad(double v) {
    const int lo = __double2loint(v), hi = __double2hiint(v);
    return __hiloint2double(__builtin_amdgcn_mov_dpp(hi, CTRL, 0xF, 0xF, true),
                            __builtin_amdgcn_mov_dpp(lo, CTRL, 0xF, 0xF, true));
}
// (v0 + v1) + (v2 + v3) over the four lanes of a quad (the four children of a
// parent: columns 4j .. 4j + 3)
__device__ __forceinline__ double quad_sum(double v) {
    v += dpp_quad<0xB1>(v);
    return v + dpp_quad<0x4E>(v);
}

__device__ __forceinline__ Frame box_frame(const double* cen, int b, double* rho) {
    const double4 c = reinterpret_cast<const double4*>(cen)[b];
    *rho = c.w;
    return make_frame(c.x, c.y, c.z);
}
}  // namespace

// Lemma 2: the parents of the boxes c0 .. c1 - 1 (one level, sibling groups of
// four) gather their children.  An empty child has a zero record.
template <int P>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2))) k_m2m(FmmCtx c, int c0, int c1) {
    __builtin_amdgcn_s_setprio(3);  // before the direct sums' waves that run beside it
    constexpr int NT = P / 4 + 1;
    const int lane = threadIdx.x, kq = lane >> 4;
    const int base = c0 + 16 * blockIdx.x, ch = min(base + (lane & 15), c1 - 1);
    const int par = c.parent[ch];
    double rho_t, rho_s;
    const Frame ft = box_frame(c.cen, par, &rho_t), fs = box_frame(c.cen, ch, &rho_s);
    const TransGeom G = trans_geom<kM2M>(fs, rho_s, ft, rho_t);
    const double* in = c.mult + (size_t)ch * (2 * P + 2);
    double re[NT], im[NT], u0;
    translate_cols<P>(in, G, kq, re, im, &u0);
    double* out = c.mult + (size_t)par * (2 * P + 2);
    const bool store = base + (lane & 15) < c1;  // whole quads
    const double cs = quad_sum(in[0] + in[1] * G.clog + 2.0 * u0), qs = quad_sum(in[1]);
    if (store && kq == 0 && (lane & 3) == 0) *reinterpret_cast<double2*>(out) = make_double2(cs, qs);
#pragma unroll
    for (int r = 0; r < NT; ++r) {
        const int l = 4 * r + kq;
        const double sr = quad_sum(re[r]), si = quad_sum(im[r]);
        if (store && (lane & 3) == (r & 3) && l >= 1 && l <= P)
            *reinterpret_cast<double2*>(out + 2 * l) = make_double2(sr, si);
    }
}

// Lemma 4: the boxes c0 .. c1 - 1 of one level take their parents' local
// expansions (boxes without targets below: left out)
template <int P>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2))) k_l2l(FmmCtx c, int c0, int c1) {
    __builtin_amdgcn_s_setprio(3);  // before the direct sums' waves that run beside it
    constexpr int NT = P / 4 + 1;
    const int lane = threadIdx.x, kq = lane >> 4;
    const int base = c0 + 16 * blockIdx.x, ch = min(base + (lane & 15), c1 - 1);
    const bool store = base + (lane & 15) < c1 && (!c.need || c.need[ch]);
    if (!any_lane(store)) return;
    const int par = c.parent[ch];
    double rho_t, rho_s;
    const Frame ft = box_frame(c.cen, ch, &rho_t), fs = box_frame(c.cen, par, &rho_s);
    const TransGeom G = trans_geom<kL2L>(fs, rho_s, ft, rho_t);
    const double* in = c.local + (size_t)par * (2 * P + 2);
    // the box's own record, loaded beside the parent's (entry 4 r + kq; entry 0
    // is C, Q; the clamp only repeats a load)
    double2* out = reinterpret_cast<double2*>(c.local + (size_t)ch * (2 * P + 2));
    double2 own[NT];
#pragma unroll
    for (int r = 0; r < NT; ++r) own[r] = out[min(4 * r + kq, P)];
    double re[NT], im[NT], u0;
    translate_cols<P>(in, G, kq, re, im, &u0);
    if (!store) return;
    if (kq == 0) {
        re[0] = in[0] + in[1] * G.clog + 2.0 * u0;
        im[0] = in[1];
    }
#pragma unroll
    for (int r = 0; r < NT; ++r)
        if (4 * r + kq <= P) out[4 * r + kq] = make_double2(own[r].x + re[r], own[r].y + im[r]);
}

void fmm_m2m(const FmmCtx& c, int c0, int c1, hipStream_t s) {
    if (c1 <= c0) return;
    const unsigned g = (unsigned)((c1 - c0 + 15) / 16);
#define L_(P) case P: k_m2m<P><<<g, 64, 0, s>>>(c, c0, c1); break;
    SFMM_DISPATCH(c.p, L_)
#undef L_
    SFMM_LAUNCH_CHECK();
}

void fmm_l2l(const FmmCtx& c, int c0, int c1, hipStream_t s) {
    if (c1 <= c0) return;
    const unsigned g = (unsigned)((c1 - c0 + 15) / 16);
#define L_(P) case P: k_l2l<P><<<g, 64, 0, s>>>(c, c0, c1); break;
    SFMM_DISPATCH(c.p, L_)
#undef L_
    SFMM_LAUNCH_CHECK();
}

}  // namespace sfmm

// Expansion arithmetic of the sFMM (Sec. 3.1-3.3, 3.6) for one box or one box
// pair, written for one GPU lane with the order P fixed at compile time so
// the coefficients live in registers.
//
// Frames.  A box centre c carries the system K_c whose zenith is c and whose
// azimuth reference is e_theta(c) (Sec. 3.1).  The base function
// z = tan(theta/2) e^{i phi} is the stereographic projection from -c,
// w = ((n - c).e_theta + i (n - c).e_phi) / (1 + n.c), with 1 + n.c computed
// as |n + c|^2 / 2 so that neither near nor antipodal points cancel.
//
// Scaled coefficients.  A box of radius R has scale rho = tan(R/2), the
// largest |w| of a point inside it.  Multipole coefficients are stored as
// A_l / rho^l and local ones as A_l rho^l, so every stored number is bounded
// by the box's mass and nothing over- or underflows down to depth 29.
//
// Translations.  Lemmas 2, 3 and 4 share one shape,
//   A'_l = ph2^l [ -(Q/l) x^l + sum_l' T_ll'(x) ph1^l' A_l' ],
//   T_ll'(x) = sum_n C(l-1,n-1) C(l',n) x^{l+l'-2n} (1+x^2)^n,
// and with the scalings folded in, T_ll' s_T^l s_S^l' factors as
//   sum_n [C(l-1,n-1) a^{l-n}] g^n [C(l',n) b^{l'-n}],
//   a = x s_T, b = x s_S, g = s_T s_S (1+x^2),
// i.e. a Taylor shift by b (right factor), a diagonal g^n, and a transposed
// Taylor shift by a (left factor).  Both shifts run in place with P(P+1)/2
// complex*real FMAs and no binomial table; a, b, g are all below ~1 for every
// pair the MACs accept, so nothing overflows.  The kernels (the FP64 M2L and
// M2M ones from order 30 up) apply the diagonal first, on the input phases
// ((g ph1)^l'), and then the shift by b/g: every
// elementary step a_j += b a_{j+1} of the shift turns into g^j a_j +=
// (b/g) g^{j+1} a_{j+1}, so D(g) T_b = T_{b/g} D(g) exactly and each
// intermediate is the old one times g^j (no new range, one multiply per
// coefficient fewer).  The n = 0 entry of the first shift is
// sum_l' b^l' ph1^l' A_l', the series part of C'.
#pragma once
#include "dd.hpp"

namespace sfmm {

constexpr double kInv4Pi = 0.079577471545947667884;  // 1 / (4 pi)
constexpr double kInv2Pi = 0.15915494309189533577;   // 1 / (2 pi)
constexpr double kLog2 = 0.69314718055994530942;
constexpr double kLog4 = 1.3862943611198906188;

// 1/x for a positive normal double: the hardware estimate refined by two
// Newton steps on the GPU (full precision), a division on the host.
SFMM_HD double recip(double x) {
#if defined(__HIP_DEVICE_COMPILE__)
    double r = __builtin_amdgcn_rcp(x);
    double e = fma(-x, r, 1.0);
    r = fma(r, e, r);
    e = fma(-x, r, 1.0);
    return fma(r, e, r);
#else
    return 1.0 / x;
#endif
}

// Natural log of a positive normal double, ~2 ulp: x = 2^e m with
// m in [1/sqrt2, sqrt2), s = (m - 1)/(m + 1), and
//   log m = 2 atanh s = 2 s (1 + s^2/3 + s^4/5 + ... + s^20/21),
// whose first omitted term is below 3e-17 relative since s^2 <= 0.0295
// (the reduction of fdlibm's e_log.c, here with the Taylor coefficients of
// atanh instead of its minimax polynomial).  e log 2 is added with the
// Cody-Waite two-word split of log 2 that fdlibm's e_log.c uses (Sun
// Microsystems, freely distributable): ln2_hi keeps 32 significant bits, so
// e ln2_hi is exact for every exponent of a double, and ln2_lo = log 2 -
// ln2_hi to double precision.  Written for the
// near-field inner loop, where the library log (a double-double algorithm
// of ~85 instructions) dominated the cost.
SFMM_HD double log_f64(double x) {
    int e;
    double m = frexp(x, &e);  // x = m 2^e, m in [1/2, 1)
    if (m < 0.70710678118654752440) {
        m *= 2.0;
        e -= 1;
    }
    const double f = m - 1.0;  // exact (Sterbenz)
    const double s = f * recip(2.0 + f);
    const double z = s * s;
    double poly = 1.0 / 21.0;
    poly = fma(poly, z, 1.0 / 19.0);
    poly = fma(poly, z, 1.0 / 17.0);
    poly = fma(poly, z, 1.0 / 15.0);
    poly = fma(poly, z, 1.0 / 13.0);
    poly = fma(poly, z, 1.0 / 11.0);
    poly = fma(poly, z, 1.0 / 9.0);
    poly = fma(poly, z, 1.0 / 7.0);
    poly = fma(poly, z, 1.0 / 5.0);
    poly = fma(poly, z, 1.0 / 3.0);
    // 2s + 2s z poly, the small part added last
    const double two_s = 2.0 * s;
    const double lm = fma(two_s * z, poly, two_s);
    const double de = (double)e;
    const double ln2_hi = 6.93147180369123816490e-01;  // top bits of log 2, e * ln2_hi exact
    const double ln2_lo = 1.90821492927058770002e-10;
    return fma(de, ln2_hi, fma(de, ln2_lo, lm));
}

// The pair loop's log and reciprocal from one table (the table-driven method
// of P. T. P. Tang, ACM TOMS 16 (1990) 378-400, with a shorter polynomial):
// x = 2^e m, m in [1/2, 1); the top 9 fraction bits of m pick c_j = 1/2 + (j +
// 1/2)/1024 and tab[j] = {1/c_j, -log(1/c_j)} (log_tab_entry), so that r =
// m/c_j - 1 (one FMA) has |r| <= 2^-10 and
//   log x = e log 2 - log(1/c_j) + log(1 + r),
// log(1 + r) = r + r^2 (-1/2 + r/3 - r^2/4 + r^3/5), first omitted term below
// 2^-62; e log 2 in log_f64's two words.  The error is absolute (near x = 1 the
// terms cancel; the sums it feeds only need that): at most 1.96e-16 of max(1,
// |log x|), 4.9e-17 in the mean square over (0, 4).  The reciprocal starts from
// the same r, 1/m = (1/c_j)(1 - r) to r^2 <= 2^-20, and one step of third order
// (d = 1 - m y, y (1 + d + d^2)) makes it 1.11e-16 at most and 4.9e-17 in the
// mean square, as two Newton steps on a hardware estimate do.  (Without that
// step, as table entry times a series in r, it was 3.3e-16 and 8.7e-17, and a
// log 2 in one word made the logs' mean square 5.8e-17.)  35 full-rate VALU
// instructions a pair; with the hardware estimate and a degree-7 series from a
// quarter of the table 39, one of which counts four.
// The Horner coefficients (the last one, -1/2, is an inline constant of the
// FMA): kernels take them as an argument, which keeps them in scalar registers.
struct LogPoly {
    double c5, c4, c3, ln2_hi, ln2_lo;  // 1/5, -1/4, 1/3, log 2
};
constexpr LogPoly kLogPoly = {1.0 / 5.0, -0.25, 1.0 / 3.0, 6.93147180369123816490e-01, 1.90821492927058770002e-10};
constexpr int kLogTab = 512;
// The table {1/c_j, -log(1/c_j)}, made by the compiler: an error of an entry is
// one of every value near c_j, so the logs are correctly rounded (with log_f64's
// they were up to an ulp off).  log c_j in two doubles, c_j = (1025 + 2 j)/2048:
// from log(1025/1024) - log 2 on, log((n + 2)/n) = 2 atanh(1/(n + 1)) a step;
// less ci c - 1 for the rounded ci = 1/c.
struct LogTab {
    double e[2 * kLogTab];
};
constexpr LogTab make_log_tab() {
    struct Two {
        double hi, lo;
        constexpr void add(double x) {
            const double s = hi + x, b = s - hi;
            lo += (hi - (s - b)) + (x - b);
            hi = s;
        }
        constexpr void add_2atanh_inv(double m) {  // 2 atanh(1/m), m > 1000
            const double x = 1.0 / m, x2 = x * x;
            lo += 2.0 * (-prod_less_1(x, m) / m) + 2.0 * x * x2 * (1.0 / 3.0 + x2 * (1.0 / 5.0 + x2 / 7.0));
            add(2.0 * x);
        }
        static constexpr double prod_less_1(double a, double b) {  // a b - 1 for a b near 1 (Dekker's product)
            const double ca = 134217729.0 * a, cb = 134217729.0 * b;
            const double ah = ca - (ca - a), al = a - ah, bh = cb - (cb - b), bl = b - bh, p = a * b;
            return (p - 1.0) + (((ah * bh - p) + ah * bl + al * bh) + al * bl);
        }
    };
    LogTab t{};
    Two l{-6.93147180559945286227e-01, -2.31904681384629955842e-17};  // -log 2
    l.add_2atanh_inv(2049.0);
    for (int j = 0; j < kLogTab; ++j) {
        const double c = (1025.0 + 2.0 * j) / 2048.0, ci = 1.0 / c;
        t.e[2 * j] = ci;
        t.e[2 * j + 1] = l.hi + (l.lo - Two::prod_less_1(ci, c));
        l.add_2atanh_inv(1026.0 + 2.0 * j);
    }
    return t;
}
#if defined(__HIP_DEVICE_COMPILE__)
static __device__ const LogTab kLogTabData = make_log_tab();
#else
static constexpr LogTab kLogTabData = make_log_tab();
#endif
SFMM_HD double2 log_tab_entry(int j) { return make_double2(kLogTabData.e[2 * j], kLogTabData.e[2 * j + 1]); }

// the table entry of a mantissa m in [1/2, 1) whose high word is hi (of the
// argument itself it would be another one's where that is subnormal)
SFMM_HD double2 log_tab_at(uint32_t hi, const double2* tab) {
    return *reinterpret_cast<const double2*>(reinterpret_cast<const char*>(tab) + (hi >> 7 & 0x1ff0u));
}

// log and reciprocal of a positive double m 2^e, m in [1/2, 1), with m's table entry t
SFMM_HD void log_recip_at(double m, int e, double2 t, const LogPoly& k, double* lg, double* inv) {
    const double r = fma(m, t.x, -1.0);
    double q = fma(k.c5, r, k.c4);
    q = fma(q, r, k.c3);
    q = fma(q, r, -0.5);
    const double de = (double)e;
    *lg = fma(de, k.ln2_hi, fma(de, k.ln2_lo, t.y + fma(r * r, q, r)));
    const double y = fma(t.x, -r, t.x);
    const double d = fma(-m, y, 1.0);
    *inv = ldexp(fma(y, fma(d, d, d), y), -e);
}

SFMM_HD void log_recip_tab(double x, const double2* tab, const LogPoly& k, double* lg, double* inv) {
    int e;
    const double m = frexp(x, &e);
    log_recip_at(m, e, log_tab_at((uint32_t)(__builtin_bit_cast(unsigned long long, m) >> 32), tab), k, lg, inv);
}

struct cplx {
    double re, im;
};
SFMM_HD cplx cmul(cplx a, cplx b) { return {a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re}; }
SFMM_HD cplx cadd(cplx a, cplx b) { return {a.re + b.re, a.im + b.im}; }
SFMM_HD cplx cconj(cplx a) { return {a.re, -a.im}; }

struct Frame {
    double c[3], et[3], ep[3];
};

// e_theta and e_phi at the centre c (never a pole for a HEALPix centre)
SFMM_HD Frame make_frame(double x, double y, double z) {
    Frame f;
    f.c[0] = x;
    f.c[1] = y;
    f.c[2] = z;
    const double rxy = sqrt(x * x + y * y);
    const double inv = 1.0 / rxy;
    f.et[0] = x * z * inv;
    f.et[1] = y * z * inv;
    f.et[2] = -rxy;
    f.ep[0] = -y * inv;
    f.ep[1] = x * inv;
    f.ep[2] = 0.0;
    return f;
}

// stereographic coordinate of n in K_c; also returns 1 + n.c
SFMM_HD cplx stereo(const Frame& f, double nx, double ny, double nz, double* one_plus_cos) {
    const double dx = nx - f.c[0], dy = ny - f.c[1], dz = nz - f.c[2];
    const double sx = nx + f.c[0], sy = ny + f.c[1], sz = nz + f.c[2];
    const double den = 0.5 * (sx * sx + sy * sy + sz * sz);
    const double inv = 1.0 / den;
    *one_plus_cos = den;
    return {(dx * f.et[0] + dy * f.et[1] + dz * f.et[2]) * inv,
            (dx * f.ep[0] + dy * f.ep[1] + dz * f.ep[2]) * inv};
}

enum TransKind { kM2M = 0, kM2L = 1, kL2L = 2 };

// Everything a translation S -> T needs besides the coefficients.
struct TransGeom {
    cplx ph1, ph2;        // phase factors applied per power on input / output
    double a, b, g;       // shift parameters of the factorised T
    double bg;            // b / g: the right shift once the diagonal g^n is applied first
    double clog;          // log cos^2(T/2) (M2M, L2L) or log sin^2(T/2) (M2L)
};

// Pair geometry from centres and scales (rho = tan(R/2)) of the source box S
// and the target box T.
template <int KIND>
SFMM_HD TransGeom trans_geom(const Frame& fs, double rho_s, const Frame& ft, double rho_t) {
    TransGeom G;
    const double dx = ft.c[0] - fs.c[0], dy = ft.c[1] - fs.c[1], dz = ft.c[2] - fs.c[2];
    const double sx = ft.c[0] + fs.c[0], sy = ft.c[1] + fs.c[1], sz = ft.c[2] + fs.c[2];
    const double dif2 = dx * dx + dy * dy + dz * dz;  // 4 sin^2(T/2)
    const double sum2 = sx * sx + sy * sy + sz * sz;  // 4 cos^2(T/2)
    // phase of T's centre seen from S, and of S's centre seen from T
    cplx e1, e2;
    if (sum2 < 1e-24) {
        // exactly antipodal centres: the geodesic leaving S along e_theta(S)
        e1 = {1.0, 0.0};
        const double u = fs.et[0] * ft.et[0] + fs.et[1] * ft.et[1] + fs.et[2] * ft.et[2];
        const double v = fs.et[0] * ft.ep[0] + fs.et[1] * ft.ep[1] + fs.et[2] * ft.ep[2];
        const double r = 1.0 / sqrt(u * u + v * v);
        e2 = {u * r, v * r};
    } else {
        const double u1 = dx * fs.et[0] + dy * fs.et[1] + dz * fs.et[2];
        const double v1 = dx * fs.ep[0] + dy * fs.ep[1] + dz * fs.ep[2];
        const double r1 = 1.0 / sqrt(u1 * u1 + v1 * v1);
        e1 = {u1 * r1, v1 * r1};
        const double u2 = -(dx * ft.et[0] + dy * ft.et[1] + dz * ft.et[2]);
        const double v2 = -(dx * ft.ep[0] + dy * ft.ep[1] + dz * ft.ep[2]);
        const double r2 = 1.0 / sqrt(u2 * u2 + v2 * v2);
        e2 = {u2 * r2, v2 * r2};
    }
    if (KIND == kM2M) {
        // Lemma 2: x = tan(T/2); s_T = 1/rho_T (multipole), s_S = rho_S
        const double t = sqrt(dif2 / sum2);
        G.ph1 = {-e1.re, e1.im};  // (-1)^l' e^{-i l' phi_T^(S)}
        G.ph2 = e2;               // e^{+i l phi_S^(T)}
        G.a = t / rho_t;
        G.b = t * rho_s;
        G.g = (rho_s / rho_t) * (1.0 + t * t);
        G.bg = t * rho_t / (1.0 + t * t);
        G.clog = log_f64(0.25 * sum2);
    } else if (KIND == kM2L) {
        // Lemma 3: x = cot(T/2); s_T = rho_T (local), s_S = rho_S
        const double c = sqrt(sum2 / dif2);
        G.ph1 = cconj(e1);  // e^{-i l' phi_T^(S)}
        G.ph2 = cconj(e2);  // e^{-i l phi_S^(T)}
        G.a = c * rho_t;
        G.b = c * rho_s;
        G.g = rho_t * rho_s * (1.0 + c * c);
        G.bg = c / (rho_t * (1.0 + c * c));
        G.clog = log_f64(0.25 * dif2);
    } else {
        // Lemma 4: x = tan(T/2); s_T = rho_T (local), s_S = 1/rho_S
        const double t = sqrt(dif2 / sum2);
        G.ph1 = e1;                  // e^{+i l' phi_T^(S)}
        G.ph2 = {-e2.re, e2.im};     // (-1)^l e^{-i l phi_S^(T)}
        G.a = t * rho_t;
        G.b = t / rho_s;
        G.g = (rho_t / rho_s) * (1.0 + t * t);
        G.bg = t / (rho_t * (1.0 + t * t));
        G.clog = log_f64(0.25 * sum2);
    }
    return G;
}

// Expansion record: e[0] = C, e[1] = Q, e[2 + 2(l-1)] = Re A_l, e[3 + 2(l-1)]
// = Im A_l (scaled).  Adds the translated expansion of `in` to acc.
template <int P>
SFMM_HD void translate_add(const double* in, const TransGeom& G, double* acc) {
    double ar[P + 1], ai[P + 1];
    const double C = in[0], Q = in[1];
    ar[0] = 0.0;
    ai[0] = 0.0;
    // diagonal g^n first, on the input phases: D(g) T_b = T_{b/g} D(g)
    const cplx pg = {G.ph1.re * G.g, G.ph1.im * G.g};
    cplx pw = pg;
#pragma unroll
    for (int l = 1; l <= P; ++l) {
        const cplx a = {in[2 * l], in[2 * l + 1]};
        const cplx v = cmul(pw, a);
        ar[l] = v.re;
        ai[l] = v.im;
        pw = cmul(pw, pg);
    }
    // right factor: Taylor shift by b/g, a[j] += (b/g) a[j+1]
#pragma unroll
    for (int i = 0; i < P; ++i) {
#pragma unroll
        for (int j = P - 1; j >= i; --j) {
            ar[j] = fma(G.bg, ar[j + 1], ar[j]);
            ai[j] = fma(G.bg, ai[j + 1], ai[j]);
        }
    }
    const double u0 = ar[0];
    // left factor: transposed Taylor shift by a on entries 1..P
#pragma unroll
    for (int i = P - 2; i >= 0; --i) {
#pragma unroll
        for (int j = i; j <= P - 2; ++j) {
            ar[j + 2] = fma(G.a, ar[j + 1], ar[j + 2]);
            ai[j + 2] = fma(G.a, ai[j + 1], ai[j + 2]);
        }
    }
    cplx pw2 = G.ph2;
    double an = G.a;
#pragma unroll
    for (int l = 1; l <= P; ++l) {
        const cplx v = {fma(-Q * (1.0 / l), an, ar[l]), ai[l]};  // 1.0 / l folds to a constant
        const cplx o = cmul(pw2, v);
        acc[2 * l] += o.re;
        acc[2 * l + 1] += o.im;
        pw2 = cmul(pw2, G.ph2);
        an *= G.a;
    }
    acc[0] += C + Q * G.clog + 2.0 * u0;
    acc[1] += Q;
}

// translate_add for one order class of a per-pair order policy: the pair's
// multipole part translated at order P, its monopole part (-(Q/l) a^l, the
// source as a point mass) completed up to the record order PO; acc holds
// 2 PO + 2 entries.
template <int P, int PO>
SFMM_HD void translate_add_po(const double* in, const TransGeom& G, double* acc) {
    translate_add<P>(in, G, acc);
    if constexpr (PO > P) {
        const double Q = in[1];
        cplx pw2 = G.ph2;
        double an = G.a;
#pragma unroll
        for (int l = 1; l <= P; ++l) {  // powers up to P
            pw2 = cmul(pw2, G.ph2);
            an *= G.a;
        }
#pragma unroll
        for (int l = P + 1; l <= PO; ++l) {
            const double v = -Q * (1.0 / l) * an;
            acc[2 * l] = fma(pw2.re, v, acc[2 * l]);
            acc[2 * l + 1] = fma(pw2.im, v, acc[2 * l + 1]);
            pw2 = cmul(pw2, G.ph2);
            an *= G.a;
        }
    }
}

// translate_add without an accumulator: in(k) gives input entry k and
// out(k, v) takes output entry k as soon as it is formed (entries 2..2P+1 in
// order, then C and Q), for kernels with one translation per lane.  Without
// the 2P + 2 accumulator registers two waves fit on a SIMD.
template <int P, class In, class Out>
SFMM_HD void translate_emit(const In& in, const TransGeom& G, const Out& out) {
    double ar[P + 1], ai[P + 1];
    const double C = in(0), Q = in(1);
    ar[0] = 0.0;
    ai[0] = 0.0;
    // from order 30 up the diagonal g^n moves in front of the right shift
    // (D(g) T_b = T_{b/g} D(g)), where it rides on the input phases: (g
    // ph1)^l.  Measured on the two-lane M2L: 3.00 -> 2.83 ms at p = 38
    // (N = 1e7); at p = 20 (N = 1e8) the folded form ran 15.5 ms against 11.2.
    constexpr bool kDiagFirst = P >= 30;
    const cplx pg = kDiagFirst ? cplx{G.ph1.re * G.g, G.ph1.im * G.g} : G.ph1;
    const double bs = kDiagFirst ? G.bg : G.b;
    cplx pw = pg;
#pragma unroll
    for (int l = 1; l <= P; ++l) {
        const cplx a = {in(2 * l), in(2 * l + 1)};
        const cplx v = cmul(pw, a);
        ar[l] = v.re;
        ai[l] = v.im;
        pw = cmul(pw, pg);
    }
#pragma unroll
    for (int i = 0; i < P; ++i) {
#pragma unroll
        for (int j = P - 1; j >= i; --j) {
            ar[j] = fma(bs, ar[j + 1], ar[j]);
            ai[j] = fma(bs, ai[j + 1], ai[j]);
        }
    }
    const double u0 = ar[0];
    if constexpr (!kDiagFirst) {
        double gn = G.g;
#pragma unroll
        for (int n = 1; n <= P; ++n) {
            ar[n] *= gn;
            ai[n] *= gn;
            gn *= G.g;
        }
    }
#pragma unroll
    for (int i = P - 2; i >= 0; --i) {
#pragma unroll
        for (int j = i; j <= P - 2; ++j) {
            ar[j + 2] = fma(G.a, ar[j + 1], ar[j + 2]);
            ai[j + 2] = fma(G.a, ai[j + 1], ai[j + 2]);
        }
    }
    cplx pw2 = G.ph2;
    double an = G.a;
#pragma unroll
    for (int l = 1; l <= P; ++l) {
        const cplx v = {fma(-Q * (1.0 / l), an, ar[l]), ai[l]};  // 1.0 / l folds to a constant
        const cplx o = cmul(pw2, v);
        out(2 * l, o.re);
        out(2 * l + 1, o.im);
        pw2 = cmul(pw2, G.ph2);
        an *= G.a;
    }
    out(0, C + Q * G.clog + 2.0 * u0);
    out(1, Q);
}

// FP32 complex numbers for the precision tier's translation (below).
struct cplxf {
    float re, im;
};
SFMM_HD cplxf cmulf(cplxf a, cplxf b) { return {a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re}; }

// The precision tier's Lemma 3 translation: the FP32 A-block (scaled,
// A[2l-2] = Re A_l, A[2l-1] = Im A_l) through the factorised map in FP32,
// with the pair geometry G computed in FP64 and rounded once; the results
// are added to acc[2P] in FP64, so the sum over an FMM-act list carries no
// FP32 rounding, and C and Q stay FP64 (accCQ).  With PO > P (a pair whose
// own order P is below the record order PO) the multipole part is cut at P
// and the monopole part, -(Q/l) a^l ph2^l, still runs to PO: acc[2 PO].
template <int P, int PO = P>
SFMM_HD void translate_add_f32_d(const float* __restrict__ A, double C, double Q, const TransGeom& G, double* acc,
                                 double* accCQ) {
    float ar[P + 1], ai[P + 1];
    ar[0] = 0.0f;
    ai[0] = 0.0f;
    const cplxf ph2 = {(float)G.ph2.re, (float)G.ph2.im};
    // diagonal g^n first, on the input phases: D(g) T_b = T_{b/g} D(g)
    const float a = (float)G.a, bg = (float)G.bg;
    const cplxf pg = {(float)(G.ph1.re * G.g), (float)(G.ph1.im * G.g)};
    cplxf pw = pg;
#pragma unroll
    for (int l = 1; l <= P; ++l) {
        const cplxf v = cmulf(pw, cplxf{A[2 * l - 2], A[2 * l - 1]});
        ar[l] = v.re;
        ai[l] = v.im;
        pw = cmulf(pw, pg);
    }
#pragma unroll
    for (int i = 0; i < P; ++i) {
#pragma unroll
        for (int j = P - 1; j >= i; --j) {
            ar[j] = fmaf(bg, ar[j + 1], ar[j]);
            ai[j] = fmaf(bg, ai[j + 1], ai[j]);
        }
    }
    const double u0 = (double)ar[0];
#pragma unroll
    for (int i = P - 2; i >= 0; --i) {
#pragma unroll
        for (int j = i; j <= P - 2; ++j) {
            ar[j + 2] = fmaf(a, ar[j + 1], ar[j + 2]);
            ai[j + 2] = fmaf(a, ai[j + 1], ai[j + 2]);
        }
    }
    const float qf = (float)Q;
    cplxf pw2 = ph2;
    float an = a;
#pragma unroll
    for (int l = 1; l <= P; ++l) {
        const cplxf v = {ar[l] - qf * (1.0f / l) * an, ai[l]};
        const cplxf o = cmulf(pw2, v);
        acc[2 * l - 2] += (double)o.re;
        acc[2 * l - 1] += (double)o.im;
        pw2 = cmulf(pw2, ph2);
        an *= a;
    }
#pragma unroll
    for (int l = P + 1; l <= PO; ++l) {
        const float v = -qf * (1.0f / l) * an;
        acc[2 * l - 2] += (double)(pw2.re * v);
        acc[2 * l - 1] += (double)(pw2.im * v);
        pw2 = cmulf(pw2, ph2);
        an *= a;
    }
    accCQ[0] += C + Q * G.clog + 2.0 * u0;
    accCQ[1] += Q;
}

// Local expansion at a point (Sec. 3.6), pole-free: psi_e and the tangent
// vector alpha_e = grad psi_e in global axes.  With f(w) = sum A_l w^l,
// psi_e = C + Q log(1 + cos theta) + 2 Re f and, in the orthonormal basis of
// the w-plane, alpha_u + i alpha_v = (1 + |w|^2) conj(f'(w)) - Q w.
template <int P>
SFMM_HD void l2p_eval(const double* e, const Frame& f, double rho, double nx, double ny, double nz,
                      double* psi, double* ax, double* ay, double* az) {
    double opc;
    const cplx w = stereo(f, nx, ny, nz, &opc);
    const double inv_rho = 1.0 / rho;
    const cplx zt = {w.re * inv_rho, w.im * inv_rho};
    // f = sum L_l zt^l by Horner from the top coefficient and g = f'(zt) =
    // sum l L_l zt^(l-1) by the companion recurrence d <- d zt + p
    cplx pv = {e[2 * P], e[2 * P + 1]}, gv = {0.0, 0.0};
#pragma unroll
    for (int l = P - 1; l >= 1; --l) {
        gv = {fma(gv.re, zt.re, fma(-gv.im, zt.im, pv.re)), fma(gv.re, zt.im, fma(gv.im, zt.re, pv.im))};
        pv = {fma(pv.re, zt.re, fma(-pv.im, zt.im, e[2 * l])), fma(pv.re, zt.im, fma(pv.im, zt.re, e[2 * l + 1]))};
    }
    gv = {fma(gv.re, zt.re, fma(-gv.im, zt.im, pv.re)), fma(gv.re, zt.im, fma(gv.im, zt.re, pv.im))};
    const cplx fv = cmul(pv, zt);
    const double C = e[0], Q = e[1];
    *psi = C + Q * log_f64(opc) + 2.0 * fv.re;
    // f'(w) = g / rho
    const double w2 = w.re * w.re + w.im * w.im;
    const double s = (1.0 + w2) * inv_rho;
    const double Ar = s * gv.re - Q * w.re;
    const double Ai = -s * gv.im - Q * w.im;
    const double inv = 1.0 / (1.0 + w2);
    const double u = w.re, v = w.im;
    // e_u = ((1+v^2-u^2) e_t - 2uv e_p - 2u c)/(1+|w|^2), e_v likewise
    const double eu_t = (1.0 + v * v - u * u) * inv, eu_p = -2.0 * u * v * inv, eu_c = -2.0 * u * inv;
    const double ev_t = -2.0 * u * v * inv, ev_p = (1.0 + u * u - v * v) * inv, ev_c = -2.0 * v * inv;
    const double at = Ar * eu_t + Ai * ev_t, ap = Ar * eu_p + Ai * ev_p, ac = Ar * eu_c + Ai * ev_c;
    *ax = at * f.et[0] + ap * f.ep[0] + ac * f.c[0];
    *ay = at * f.et[1] + ap * f.ep[1] + ac * f.c[1];
    *az = at * f.et[2] + ap * f.ep[2] + ac * f.c[2];
}

// Multipole expansion (Lemma 1 form) of a source box evaluated at a point n
// far from it: psi = C + Q log(1 - cos theta) + 2 Re sum A_l w^-l and its
// tangent gradient.  With zeta = rho / w, f = sum Ah_l zeta^l and
// g = sum l Ah_l zeta^l (Ah the scaled coefficients), the w-plane gradient of
// 2 Re f is -2 conj(g / w) and that of Q log(1 - cos) = Q log(2|w|^2/(1+|w|^2))
// is 2 Q w / (|w|^2 (1 + |w|^2)), so
//   alpha_u + i alpha_v = (Q - (1 + |w|^2) conj(g)) / conj(w).
// In three parts, which the Hessian below shares: the point in the box's frame,
// the series, and what follows from its values.
struct M2PPoint {
    cplx w, zt;  // zt = rho / w
    double w2, iw2, omc;  // |w|^2, its reciprocal, 1 - cos theta
};

SFMM_HD M2PPoint m2p_point(const Frame& f, double rho, double nx, double ny, double nz) {
    M2PPoint q;
    double opc;
    q.w = stereo(f, nx, ny, nz, &opc);
    const double dx = nx - f.c[0], dy = ny - f.c[1], dz = nz - f.c[2];
    q.omc = 0.5 * (dx * dx + dy * dy + dz * dz);
    q.w2 = q.w.re * q.w.re + q.w.im * q.w.im;
    q.iw2 = recip(q.w2);
    q.zt = {rho * q.w.re * q.iw2, -rho * q.w.im * q.iw2};
    return q;
}

// a z + b
SFMM_HD cplx horner_step(cplx a, cplx z, cplx b) {
    return {fma(a.re, z.re, fma(-a.im, z.im, b.re)), fma(a.re, z.im, fma(a.im, z.re, b.im))};
}

// h(z) = sum_l A_l z^l at z = zt: pv = h / z, dv = h' and, with HESS, d1 = (h /
// z)' and ev = (h / z)'' / 2.  Horner from the top coefficient, the derivatives
// by companion recurrences d <- d z + p (two FMAs per real part, no l factors).
template <int P, bool HESS>
SFMM_HD void m2p_series(const double* __restrict__ e, cplx zt, cplx* pv, cplx* dv, cplx* d1, cplx* ev) {
    cplx p = {e[2 * P], e[2 * P + 1]}, d = {0.0, 0.0}, h = {0.0, 0.0};
#pragma unroll 6
    for (int l = P - 1; l >= 1; --l) {
        if (HESS) h = horner_step(h, zt, d);
        d = horner_step(d, zt, p);
        p = horner_step(p, zt, cplx{e[2 * l], e[2 * l + 1]});
    }
    *pv = p;
    *dv = horner_step(d, zt, p);
    if (HESS) {
        *d1 = d;
        *ev = h;
    }
}

SFMM_HD void m2p_finish(double C, double Q, const Frame& f, const M2PPoint& q, cplx pv, cplx dv, double* psi,
                        double* ax, double* ay, double* az) {
    const cplx w = q.w, F = cmul(pv, q.zt), G = cmul(dv, q.zt);  // G = z h'
    *psi = C + Q * log_f64(q.omc) + 2.0 * F.re;
    // (Q - (1+|w|^2) conj(G)) / conj(w) = (Q - s conj(G)) * w / |w|^2
    const double s = 1.0 + q.w2;
    const cplx num = {Q - s * G.re, s * G.im};
    const cplx A = {(num.re * w.re - num.im * w.im) * q.iw2, (num.re * w.im + num.im * w.re) * q.iw2};
    const double inv = recip(s);
    const double u = w.re, v = w.im;
    const double eu_t = (1.0 + v * v - u * u) * inv, eu_p = -2.0 * u * v * inv, eu_c = -2.0 * u * inv;
    const double ev_t = -2.0 * u * v * inv, ev_p = (1.0 + u * u - v * v) * inv, ev_c = -2.0 * v * inv;
    const double at = A.re * eu_t + A.im * ev_t, ap = A.re * eu_p + A.im * ev_p, ac = A.re * eu_c + A.im * ev_c;
    *ax = at * f.et[0] + ap * f.ep[0] + ac * f.c[0];
    *ay = at * f.et[1] + ap * f.ep[1] + ac * f.c[1];
    *az = at * f.et[2] + ap * f.ep[2] + ac * f.c[2];
}

template <int P>
SFMM_HD void m2p_eval(const double* __restrict__ e, const Frame& f, double rho, double nx, double ny, double nz,
                      double* psi, double* ax, double* ay, double* az) {
    const M2PPoint q = m2p_point(f, rho, nx, ny, nz);
    cplx pv, dv;
    m2p_series<P, false>(e, q.zt, &pv, &dv, nullptr, nullptr);
    m2p_finish(e[0], e[1], f, q, pv, dv, psi, ax, ay, az);
}


// ---------------------------------------------------------------- Hessian
// The Hessian of Sec. 2.2 (second covariant derivatives of psi in the basis
// e_theta, e_phi of the target).  In the stereographic coordinate w = u + iv
// of a box frame the sphere's metric is conformal, (2 / D)^2 |dw|^2 with
// D = 1 + |w|^2, and the covariant Hessian of psi in the orthonormal basis
// (e_u, e_v) of the w-plane is
//   H_uu + H_vv = (D^2 / 4) Laplacian_w psi,
//   H_uu - H_vv - 2i H_uv = Z = D^2 (psi_ww - 2 sigma_w psi_w),
// with psi_w = d psi / dw, sigma = log(2 / D) (so sigma_w = -conj(w) / D).
// For the local form psi = C + Q log(1 + cos) + 2 Re f(w), f = sum A_l w^l:
//   Z = D^2 f'' + 2 conj(w) D f' - Q conj(w)^2,   trace -Q;
// for the multipole form psi = C + Q log(1 - cos) + 2 Re f(w), f = sum A_l
// w^-l:
//   Z = D^2 f'' + 2 conj(w) D f' - Q / w^2,       trace -Q.
// Both are regular at w = 0 (the local form at a box centre) and need no
// angle.  The (e_u, e_v) components are then turned into the target's
// (e_theta, e_phi) ones.

// e_theta, e_phi of the target n (phi = 0 at an exact pole)
SFMM_HD void target_basis(double nx, double ny, double nz, double* et, double* ep) {
    const double rxy = sqrt(nx * nx + ny * ny);
    const double cph = rxy > 0.0 ? nx / rxy : 1.0, sph = rxy > 0.0 ? ny / rxy : 0.0;
    et[0] = nz * cph;
    et[1] = nz * sph;
    et[2] = -rxy;
    ep[0] = -sph;
    ep[1] = cph;
    ep[2] = 0.0;
}

// (H_uu, H_uv, H_vv) in the w-plane basis of frame f at w -> (H_tt, H_tp,
// H_pp) in the basis et, ep of the target
SFMM_HD void hess_to_target(const Frame& f, cplx w, double huu, double huv, double hvv, const double* et,
                            const double* ep, double* h) {
    const double u = w.re, v = w.im;
    const double inv = 1.0 / (1.0 + u * u + v * v);
    const double eu_t = (1.0 + v * v - u * u) * inv, eu_p = -2.0 * u * v * inv, eu_c = -2.0 * u * inv;
    const double ev_t = -2.0 * u * v * inv, ev_p = (1.0 + u * u - v * v) * inv, ev_c = -2.0 * v * inv;
    double eu[3], ev[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        eu[d] = eu_t * f.et[d] + eu_p * f.ep[d] + eu_c * f.c[d];
        ev[d] = ev_t * f.et[d] + ev_p * f.ep[d] + ev_c * f.c[d];
    }
    const double tu = et[0] * eu[0] + et[1] * eu[1] + et[2] * eu[2];
    const double tv = et[0] * ev[0] + et[1] * ev[1] + et[2] * ev[2];
    const double pu = ep[0] * eu[0] + ep[1] * eu[1] + ep[2] * eu[2];
    const double pv = ep[0] * ev[0] + ep[1] * ev[1] + ep[2] * ev[2];
    h[0] = tu * tu * huu + 2.0 * tu * tv * huv + tv * tv * hvv;
    h[1] = tu * pu * huu + (tu * pv + tv * pu) * huv + tv * pv * hvv;
    h[2] = pu * pu * huu + 2.0 * pu * pv * huv + pv * pv * hvv;
}

// l2p_eval and the Hessian h[3] of the local expansion at the target
// (et, ep its basis)
template <int P>
SFMM_HD void l2p_eval_hess(const double* e, const Frame& f, double rho, double nx, double ny, double nz,
                           const double* et, const double* ep, double* psi, double* ax, double* ay, double* az,
                           double* h) {
    l2p_eval<P>(e, f, rho, nx, ny, nz, psi, ax, ay, az);
    double opc;
    const cplx w = stereo(f, nx, ny, nz, &opc);
    const double inv_rho = 1.0 / rho;
    const cplx zt = {w.re * inv_rho, w.im * inv_rho};
    // Horner for q(z) = sum L_l z^(l-1) with its first derivative dv and
    // half its second ev; then g = (z q)' and k = (z q)'' = 2 (dv + z ev)
    cplx pv = {e[2 * P], e[2 * P + 1]}, dv = {0.0, 0.0}, ev = {0.0, 0.0};
#pragma unroll
    for (int l = P - 1; l >= 1; --l) {
        ev = cadd(cmul(ev, zt), dv);
        dv = cadd(cmul(dv, zt), pv);
        pv = cadd(cmul(pv, zt), cplx{e[2 * l], e[2 * l + 1]});
    }
    const cplx g = cadd(cmul(dv, zt), pv);
    const cplx k = cmul(cplx{2.0, 0.0}, cadd(dv, cmul(zt, ev)));
    const double Q = e[1];
    const double D = 1.0 + w.re * w.re + w.im * w.im;
    const cplx wc = {w.re, -w.im};
    // Z = D^2 f'' + 2 conj(w) D f' - Q conj(w)^2, f' = g / rho, f'' = k / rho^2
    const cplx t1 = cmul(cplx{D * D * inv_rho * inv_rho, 0.0}, k);
    const cplx t2 = cmul(cplx{2.0 * D * inv_rho, 0.0}, cmul(wc, g));
    const cplx wc2 = cmul(wc, wc);
    const cplx Z = {t1.re + t2.re - Q * wc2.re, t1.im + t2.im - Q * wc2.im};
    hess_to_target(f, w, 0.5 * (-Q + Z.re), -0.5 * Z.im, 0.5 * (-Q - Z.re), et, ep, h);
}

// The Hessian h[3] of a source box's multipole expansion at the target (et, ep
// its basis) from m2p_series: with zeta = rho / w and h(zeta) = sum Ah_l
// zeta^l, f' = -G / w and f'' = K / w^2, G = sum l Ah_l zeta^l = zeta h', K =
// sum l (l + 1) Ah_l zeta^l = zeta^2 h'' + 2 G, h'' = 2 (d1 + zeta ev).
SFMM_HD void m2p_finish_hess(double Q, const Frame& f, const M2PPoint& q, cplx dv, cplx d1, cplx ev,
                             const double* et, const double* ep, double* h) {
    const cplx w = q.w, zt = q.zt;
    const cplx iw = {w.re * q.iw2, -w.im * q.iw2};  // 1 / w
    const cplx F2 = cmul(cplx{2.0, 0.0}, horner_step(ev, zt, d1));
    const cplx G = cmul(zt, dv);
    const cplx z2 = cmul(zt, zt);
    const cplx K = cadd(cmul(z2, F2), cmul(cplx{2.0, 0.0}, G));
    const double D = 1.0 + q.w2;
    const cplx wc = {w.re, -w.im};
    const cplx iw2c = cmul(iw, iw);  // 1 / w^2
    // Z = D^2 K / w^2 - 2 conj(w) D G / w - Q / w^2
    const cplx a = cmul(cplx{D * D, 0.0}, cmul(K, iw2c));
    const cplx b = cmul(cplx{2.0 * D, 0.0}, cmul(wc, cmul(G, iw)));
    const cplx Z = {a.re - b.re - Q * iw2c.re, a.im - b.im - Q * iw2c.im};
    hess_to_target(f, w, 0.5 * (-Q + Z.re), -0.5 * Z.im, 0.5 * (-Q - Z.re), et, ep, h);
}

// m2p_eval and the Hessian, from one pass over the series: 12 FMAs a
// coefficient (two passes, of 8 and 12: 175 -> 119 us in k_m2p for the shear of
// 1e6 sources at 196,608 targets, p = 38).
template <int P>
SFMM_HD void m2p_eval_hess(const double* __restrict__ e, const Frame& f, double rho, double nx, double ny,
                           double nz, const double* et, const double* ep, double* psi, double* ax, double* ay,
                           double* az, double* h) {
    const M2PPoint q = m2p_point(f, rho, nx, ny, nz);
    cplx pv, dv, d1, ev;
    m2p_series<P, true>(e, q.zt, &pv, &dv, &d1, &ev);
    m2p_finish(e[0], e[1], f, q, pv, dv, psi, ax, ay, az);
    m2p_finish_hess(e[1], f, q, dv, d1, ev, et, ep, h);
}

}  // namespace sfmm

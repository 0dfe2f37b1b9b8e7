// Near field (the direct acts of Sec. 3.3-3.4): for every target in a leaf T,
// the sum of the Green's function and its tangent gradient over the particles
// of T's close leaves.
//
// At planning time each direct-act list is split in two (near_lists):
//   * a close leaf S whose centre is more than R_S / x from every target of
//     T (and that holds enough particles for it to pay) is taken through its
//     own multipole expansion (Lemma 1) at each target: k_m2p.  By Eq.
//     MUL_ERR the truncation there is below (Q~/2pi) x^(p+1)/((p+1)(1-x));
//     x is at most 1/3 and makes x^(p+1) at most 1e-4 times the tolerance of
//     order p (m2p_ratio).  The split is only made for p >= 12 and for leaves
//     with at least p/4 + 2 particles.  Big leaves of sparse regions next to
//     dense clumps are where it matters: their targets otherwise meet every
//     particle of the clump directly.
//   * every other close leaf is summed particle by particle: k_p2p.
//
// k_p2p: a wave (or, where there are few, a workgroup of four) owns one target
// leaf (or a segment of its list) and takes its targets in groups of ng <= 64,
// TB targets per lane (two in FP64, one in the precision tier and for leaves
// with few targets) and teams of L = floor(64 / ceil(ng / TB)) lanes.  The close leaves' particle ranges are concatenated into one
// flat index space (wave prefix sum of their counts, 64 entries at a time);
// each tile of 128 particles is decoded once (binary search by lane shuffles)
// and staged in LDS, and lane r of a team takes particles r, r + L, ... of the tile.  The partial sums stay in registers
// across all tiles; at the end of the group they are added over lanes and
// waves in a fixed order through LDS.  No floating-point atomics: the result
// is bitwise reproducible.
//
// Load balance: a leaf of a sparse region next to a dense clump can have
// thousands of close leaves (every clump leaf fails the MAC against a big
// leaf).  Each leaf's two lists are cut into segments of at most kSegNear /
// far_segment() entries; a workgroup takes one (leaf, segment) item, items are
// launched heaviest first, and a leaf cut into several segments writes its
// per-segment results to a partial buffer that k_near_reduce adds up in
// segment order (so the result stays bitwise reproducible).
//
// Per pair, with d = n_t - n_s, psi gets (q/4pi)(log(|d|^2/4) + 1) (Eq.
// GRE_FUN plus the zero-mean share) and alpha gets (q/2pi) d/|d|^2, projected
// on the tangent plane once per target.  A particle at exactly the target
// position keeps only its q/(4pi).  Per target only four sums are kept:
//   S = sum q log|d|^2   (log 4 in place of the log for a coincident particle)
//   V = sum q d/|d|^2    (d = 0 there, so nothing is added)
// and with Q_near = sum q over the summed leaves (from their Lemma 1 Q),
//   4 pi psi_near = S + (1 - log 4) Q_near.
#include "common.hpp"
#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <type_traits>
#include "expand.hpp"

namespace sfmm {

constexpr int kTile = 128;  // particles staged in LDS per tile

static unsigned nblk(int64_t n, int b) { return (unsigned)((n + b - 1) / b > 0 ? (n + b - 1) / b : 1); }

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// A close leaf S is evaluated through its Lemma 1 expansion at the targets
// of T when every target is beyond ratio R_S from its centre, ratio = 1 / x
// with the truncation term x^(p+1) at most 1e-4 tau_p (tau_p: the tolerance
// that gives order p by the order policy, 4 times its calibrated error), and
// at least 3: ratio 3 down to p = 21, 3.2 at p = 18, 4.2 at p = 12.  And when S holds at
// least p/4 + 2 particles (measured at p = 36: lower ratios or a higher count
// move more work than they save).
double m2p_ratio(int p) {
    const double tau = 4.0 * order_calibrated_error(p);
    const double x = std::min(1.0 / 3.0, std::pow(1e-4 * tau, 1.0 / (p + 1)));
    return 1.0 / x;
}
int m2p_min_count(int p) { return (p + 8 + 3) / 4; }  // ceil(p/4 + 2)

// Expansions per item when the caller sets no length.  A lane evaluates its
// target's expansions one after another, so a launch lasts at least as long
// as its longest segment: 128 expansions are 100-190 us at p = 20-38, where
// all items of a small plan together are a few us of work.  Short segments
// cost partial sums and their addition, which a launch that fills the chip
// many times over does not get back.  k_m2p + k_near_reduce, us, segments of
// 128 / 64 / 32 / 16:
//   5e4 sources, 3,200 leaves, p = 20   118 /  103 /  60 /  40
//   3e5, 6,900 leaves, p = 20           130 /  73 /  49 /  40
//   2.5e5, 6,100 leaves, p = 38         193 / 105 /  68 /  62   (with the Hessian)
//   1e6, 27,000 leaves, p = 38          240 / 192 / 207 / 218
//   1e7, 174,000 leaves, p = 38        1069 / 1156 / 1232 / 1345
// Many targets to a leaf fill the chip with groups of 64 instead
// (target_groups), and their partial slots would grow with them: long
// segments from 64 targets a leaf up.
int far_segment(int leaves, int64_t m) {
    if (m > 64 * (int64_t)leaves) return kSegFar;
    return leaves < 16384 ? 16 : leaves < 65536 ? 64 : kSegFar;
}

// Workgroups that share an item's groups of 64 targets (the grid's y): as
// many as the average item has groups.  With the groups one after another a
// plan of few leaves and many targets ran on few waves: 10,000 sources and 1e6 targets
// 9.9 -> 0.9 ms of direct sums and 1.65 -> 0.10 of expansions (p = 38)
static unsigned target_groups(int64_t m, int items) {
    return (unsigned)std::min<int64_t>(64, m / (64 * (int64_t)items) + 1);
}

// ------------------------------------------------------------ work per box
// Work of each box: pairs[T] = tcount[T] * (particles of the near leaves),
// evals[T] = tcount[T] * (far leaves)
__global__ void k_near_work(const int* __restrict__ count, const int* __restrict__ off,
                            const int* __restrict__ nn, const int* __restrict__ src,
                            const int* __restrict__ tcount, int nbox, long long* __restrict__ pairs,
                            long long* __restrict__ evals) {
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= nbox) return;
    long long ns = 0;
    int nf = 0;
    if (tcount[b] > 0 && off[b + 1] > off[b]) {  // nn is set for these
        for (int k = off[b]; k < off[b] + nn[b]; ++k) ns += count[src[k]];
        nf = off[b + 1] - off[b] - nn[b];
    }
    pairs[b] = ns * (long long)tcount[b];
    evals[b] = (long long)nf * (long long)tcount[b];
}

void near_work(const int* count, const int* off, const int* nn, const int* src, const int* tcount, int nbox,
               long long* pairs, long long* evals, hipStream_t s) {
    if (nbox <= 0) return;
    k_near_work<<<nblk(nbox, 256), 256, 0, s>>>(count, off, nn, src, tcount, nbox, pairs, evals);
    SFMM_LAUNCH_CHECK();
}

// ------------------------------------------------------------ work items
// Leaf i of the list tl has two lists in one CSR run: nn[T] entries for the
// direct sum, then the entries for the expansions.  Per kind: ceil(K / seg)
// items, and for a leaf cut into several of them as many times tcount partial
// slots (2^31 stands for more) and one reduce record.  cnt [6][ntl]: items,
// slots, reduce records of the first kind, then of the second.
__global__ void k_item_count(const int* __restrict__ tl, int ntl, const int* __restrict__ off,
                             const int* __restrict__ nn, const int* __restrict__ tcount, int seg_near, int seg_far,
                             int* __restrict__ cnt) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= ntl) return;
    const int T = tl[i], n = off[T + 1] - off[T], nt = tcount[T];
    const int k[2] = {n > 0 ? nn[T] : 0, n > 0 ? n - nn[T] : 0}, seg[2] = {seg_near, seg_far};
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int ns = (k[q] + seg[q] - 1) / seg[q];
        cnt[(size_t)(3 * q + 0) * ntl + i] = ns;
        cnt[(size_t)(3 * q + 1) * ntl + i] = ns > 1 ? (int)min((int64_t)ns * nt, (int64_t)1 << 31) : 0;
        cnt[(size_t)(3 * q + 2) * ntl + i] = ns > 1 ? 1 : 0;
    }
}

// Items (box, first entry, end entry, partial slot base or -1), the direct
// sums' first, and the reduce records (box, segments, base)
__global__ void k_item_emit(const int* __restrict__ tl, int ntl, const int* __restrict__ off,
                            const int* __restrict__ nn, const int* __restrict__ tcount, int seg_near, int seg_far,
                            const int* __restrict__ pos, int n_near, int red_near, int4* __restrict__ items,
                            int4* __restrict__ red) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= ntl) return;
    const int T = tl[i], nt = tcount[T], k0 = off[T], k2 = off[T + 1];
    if (k2 == k0) return;
    const int k1 = k0 + nn[T];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int ka = q ? k1 : k0, kb = q ? k2 : k1, seg = q ? seg_far : seg_near;
        const int ns = (kb - ka + seg - 1) / seg;
        const int at = pos[(size_t)(3 * q) * ntl + i] + (q ? n_near : 0), slot = pos[(size_t)(3 * q + 1) * ntl + i];
        for (int sg = 0; sg < ns; ++sg)
            items[at + sg] = make_int4(T, ka + sg * seg, min(ka + (sg + 1) * seg, kb), ns > 1 ? slot + sg * nt : -1);
        if (ns > 1) red[pos[(size_t)(3 * q + 2) * ntl + i] + (q ? red_near : 0)] = make_int4(T, ns, slot, 0);
    }
}

// Sort key of each item: direct sums (the first n_near) before expansions,
// then by the leading zeros of the work, targets x particles (targets x
// entries for expansions), heaviest power-of-two bucket first (a wave per
// item: its lanes sum the particle counts of the segment)
__global__ void k_item_keys(const int4* __restrict__ items, int n, int n_near, const int* __restrict__ src,
                            const int* __restrict__ count, const int* __restrict__ tcount,
                            uint64_t* __restrict__ keys, uint32_t* __restrict__ vals) {
    const int i = (int)((blockIdx.x * (int64_t)blockDim.x + threadIdx.x) >> 6);
    const int lane = threadIdx.x & 63;
    if (i >= n) return;  // uniform across the wave
    const int4 it = items[i];
    long long w = it.z - it.y;
    if (i < n_near) {
        long long part = 0;
        for (int k = it.y + lane; k < it.z; k += 64) part += count[src[k]];
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) part += __shfl_xor(part, o, 64);
        w = part;
    }
    if (lane != 0) return;
    w *= tcount[it.x];
    keys[i] = (i < n_near ? 0u : 128u) | (w > 0 ? (unsigned)__clzll(w) : 127u);
    vals[i] = (uint32_t)i;
}

__global__ void k_gather_items(const int4* __restrict__ in, const uint32_t* __restrict__ idx, int n,
                               int4* __restrict__ out) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) out[i] = in[idx[i]];
}

// Most partial slots of either kind.  SFMM_SLOT_LIMIT lowers it (for tests of
// the refusal).
static int64_t slot_limit() {
    const char* v = std::getenv("SFMM_SLOT_LIMIT");
    return v ? std::max(0L, std::min(0x7fffffffL, std::strtol(v, nullptr, 10))) : 0x7fffffffL;
}

void build_items(const int* tl, int ntl, const int* off, const int* nn, const int* src, const int* count,
                 const int* tcount, int seg_near, int seg_far, int64_t slots_room, NearWork& out, int* pin,
                 hipStream_t s) {
    out.near = WorkItems();
    out.far = WorkItems();
    if (ntl <= 0) return;
    DVec<int> cnt, pos;
    cnt.resize(6 * (size_t)ntl);
    pos.resize(6 * (size_t)ntl);
    auto tally = [&]() {
        k_item_count<<<nblk(ntl, 256), 256, 0, s>>>(tl, ntl, off, nn, tcount, seg_near, seg_far, cnt.data());
        SFMM_LAUNCH_CHECK();
        scan_excl_i32_n(cnt.data(), pos.data(), 6, ntl, pin, s);
        SFMM_HIP(hipStreamSynchronize(s));
    };
    tally();
    // the totals as they are, also past 2^31 - 1 (add_sat)
    auto slots = [&](int q) { return (int64_t)(uint32_t)pin[3 * q + 1]; };
    if (seg_far < kSegFar && slots(0) + slots(1) > slots_room) {
        seg_far = kSegFar;
        tally();
    }
    // a slot's number is a 32-bit one; items and reduce records are no more
    // than the lists' entries
    const int64_t lim = slot_limit();
    if (slots(0) > lim || slots(1) > lim) throw Error(ST_INVALID_ARG, "near-field partial sums too large");
    const int n_near = pin[0], n = pin[0] + pin[3], red_near = pin[2];
    out.items.resize(std::max(n, 1));
    out.red.resize(std::max(pin[2] + pin[5], 1));
    out.part.resize(4 * (size_t)std::max<int64_t>(slots(0) + slots(1), 1));
    out.near.items = out.items.data();
    out.near.red = out.red.data();
    out.near.part = out.part.data();
    out.near.n = pin[0];
    out.near.nslot = pin[1];
    out.near.nred = pin[2];
    out.near.leaves = out.far.leaves = ntl;
    out.far.items = out.items.data() + n_near;
    out.far.red = out.red.data() + red_near;
    out.far.part = out.part.data() + 4 * (size_t)pin[1];
    out.far.n = pin[3];
    out.far.nslot = pin[4];
    out.far.nred = pin[5];
    if (n == 0) return;
    DVec<int4> raw;
    DVec<uint64_t> keys;
    DVec<uint32_t> vals;
    raw.resize(n);
    keys.resize(n);
    vals.resize(n);
    k_item_emit<<<nblk(ntl, 256), 256, 0, s>>>(tl, ntl, off, nn, tcount, seg_near, seg_far, pos.data(), n_near,
                                               red_near, raw.data(), out.red.data());
    SFMM_LAUNCH_CHECK();
    k_item_keys<<<nblk(64 * (int64_t)n, 256), 256, 0, s>>>(raw.data(), n, n_near, src, count, tcount, keys.data(),
                                                           vals.data());
    SFMM_LAUNCH_CHECK();
    radix_sort_u64(keys.data(), vals.data(), n, 8, s);
    k_gather_items<<<nblk(n, 256), 256, 0, s>>>(raw.data(), vals.data(), n, out.items.data());
    SFMM_LAUNCH_CHECK();
}

// Adds the per-segment results of every box cut into several items, in
// segment order: a workgroup per box (or several, groups of 64 targets side by
// side), lanes over its targets.  Bound by the latency of its loads where a box
// has thousands of segments: eight segments' loads are under way at once (one
// after another, 6,250 segments took 9.3 ms, now 0.2).
template <bool HESS>
__global__ void __launch_bounds__(64) k_near_reduce(const int4* __restrict__ red, const int* __restrict__ tfirst,
                                                   const int* __restrict__ tcount,
                                                   const double* __restrict__ part, double* __restrict__ near,
                                                   double* __restrict__ hess, int64_t m) {
    constexpr int NV = HESS ? 7 : 4, ST = HESS ? 8 : 4;
    const int4 r = red[blockIdx.x];
    const int T = r.x, ns = r.y, base = r.z;
    const int t0 = tfirst[T], nt = tcount[T];
    for (int t = blockIdx.y * 64 + threadIdx.x; t < nt; t += 64 * gridDim.y) {
        double v[NV];
#pragma unroll
        for (int k = 0; k < NV; ++k) v[k] = 0.0;
        const double* q = part + ST * ((size_t)base + t);
        const size_t step = ST * (size_t)nt;
        constexpr int U = 8;
        double x[U][NV];
        int sg = 0;
        for (; sg + U <= ns; sg += U, q += U * step) {
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int k = 0; k < NV; ++k) x[u][k] = q[u * step + k];
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int k = 0; k < NV; ++k) v[k] += x[u][k];
        }
        if (sg < ns) {  // the last fewer than eight, the very last loaded again past the end
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int k = 0; k < NV; ++k) x[u][k] = q[min(u, ns - 1 - sg) * step + k];
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (sg + u >= ns) break;
#pragma unroll
                for (int k = 0; k < NV; ++k) v[k] += x[u][k];
            }
        }
        const int64_t o = t0 + t;
        near[o] += v[0];
        near[m + o] += v[1];
        near[2 * m + o] += v[2];
        near[3 * m + o] += v[3];
        if constexpr (HESS) {
            hess[o] += v[4];
            hess[m + o] += v[5];
            hess[2 * m + o] += v[6];
        }
    }
}

// psi and alpha contributions of one target: straight to its near field (near
// [4][m], plan order), or to its slot of the partial buffer
__device__ __forceinline__ void emit_target(int slot, int64_t i, double ps, double a0, double a1, double a2,
                                            double* __restrict__ part, double* __restrict__ near, int64_t m) {
    if (slot < 0) {
        near[i] += ps;
        near[m + i] += a0;
        near[2 * m + i] += a1;
        near[3 * m + i] += a2;
    } else {
        double* q = part + 4 * (size_t)slot;
        q[0] = ps;
        q[1] = a0;
        q[2] = a1;
        q[3] = a2;
    }
}

// the same with the Hessian h[3] (slots of 8 doubles)
__device__ __forceinline__ void emit_target_hess(int slot, int64_t i, double ps, double a0, double a1, double a2,
                                                 const double* h, double* __restrict__ part,
                                                 double* __restrict__ near, double* __restrict__ hess, int64_t m) {
    if (slot < 0) {
        emit_target(-1, i, ps, a0, a1, a2, part, near, m);
        hess[i] += h[0];
        hess[m + i] += h[1];
        hess[2 * m + i] += h[2];
    } else {
        double* q = part + 8 * (size_t)slot;
        q[0] = ps;
        q[1] = a0;
        q[2] = a1;
        q[3] = a2;
        q[4] = h[0];
        q[5] = h[1];
        q[6] = h[2];
    }
}

// ------------------------------------------------------------ direct sums
// Pair terms of one lane over one LDS tile.  FP64: coordinates as stored.
// FP32 (precision tier): every coordinate is a two-float pair hi + lo
// (hi = float(x), lo = float(x - hi)), so d = (t_hi - s_hi) + (t_lo - s_lo)
// keeps ~1e-7 relative accuracy for close points where plain FP32 positions
// would lose all digits of d; log and reciprocal are the hardware FP32
// instructions, and each tile's FP32 partial sums (at most 256 terms) are
// added to FP64 running sums.  The log terms, all of one sign, are summed
// with Kahan compensation; the deflection terms largely cancel and are not.
struct TileF32 {
    float4 hi[kTile];  // x, y, z, q
    float4 lo[kTile];  // x, y, z low parts
};

__device__ __forceinline__ void tile_store(TileF32& t, int k, double4 v) {
    const float xh = (float)v.x, yh = (float)v.y, zh = (float)v.z;
    t.hi[k] = make_float4(xh, yh, zh, (float)v.w);
    t.lo[k] = make_float4((float)(v.x - (double)xh), (float)(v.y - (double)yh), (float)(v.z - (double)zh), 0.0f);
}

// Near-particle model inside a profile (u = |d|^2/4 < t): log(4u) of the
// point mass is replaced by log(4t) - I(u/t) and the deflection weight q/|d|^2
// by (q/4)(2/t - v/t - 1)/(1 - u) (both finite at u = 0); see NpmK.
template <typename R>
__device__ __forceinline__ R npm_interior_log(R v, R t, R ln4t, int nterms) {
    // I(v) = sum_k t^k [(2 - t)(1 - v^(k+1))/(k+1) - (1 - v^(k+2))/(k+2)]
    R sum = 0, tk = 1, vk1 = v, vk2 = v * v;
    for (int k = 0; k < nterms; ++k) {
        sum += tk * ((2 - t) * (1 - vk1) / (R)(k + 1) - (1 - vk2) / (R)(k + 2));
        tk *= t;
        vk1 *= v;
        vk2 *= v;
    }
    return ln4t - sum;
}

template <bool NPM>
__device__ __forceinline__ void tile_pairs(const TileF32& t, const NpmK& nk, int r, int L, int tn, double ax, double ay, double az, double& p0, double& p1,
                                           double& p2, double& p3) {
    const float axh = (float)ax, ayh = (float)ay, azh = (float)az;
    const float axl = (float)(ax - (double)axh), ayl = (float)(ay - (double)ayh), azl = (float)(az - (double)azh);
    constexpr float kLn2f = 0.693147180559945309f, kLog4f = 1.38629436111989061f;
    float f0 = 0.0f, c0 = 0.0f, f1 = 0.0f, f2 = 0.0f, f3 = 0.0f;
    for (int j = r; j < tn; j += L) {
        const float4 h = t.hi[j], l = t.lo[j];
        const float dx = (axh - h.x) + (axl - l.x);
        const float dy = (ayh - h.y) + (ayl - l.y);
        const float dz = (azh - h.z) + (azl - l.z);
        const float d2 = dx * dx + dy * dy + dz * dz;
        const bool coinc = d2 == 0.0f;
        const float r2 = coinc ? 1.0f : d2;
        float lg = coinc ? kLog4f : __builtin_amdgcn_logf(r2) * kLn2f;
        float wi = h.w * __builtin_amdgcn_rcpf(r2);
        if constexpr (NPM) {
            if (d2 < (float)nk.four_t) {
                const float u = 0.25f * d2, v = u * (float)nk.inv_t;
                lg = npm_interior_log(v, (float)nk.t, (float)nk.ln4t, nk.nterms);
                wi = h.w * 0.25f * (2.0f * (float)nk.inv_t - v * (float)nk.inv_t - 1.0f) / (1.0f - u);
            }
        }
        // the log terms all have one sign and grow the sum to ~100 times
        // each: Kahan-compensated (c0 carries the lost low part)
        const float y = fmaf(h.w, lg, -c0);
        const float tt = f0 + y;
        c0 = (tt - f0) - y;
        f0 = tt;
        f1 = fmaf(wi, dx, f1);
        f2 = fmaf(wi, dy, f2);
        f3 = fmaf(wi, dz, f3);
    }
    p0 += (double)f0 - (double)c0;
    p1 += (double)f1;
    p2 += (double)f2;
    p3 += (double)f3;
}

// Pair terms with the Hessian of Sec. 2.2: per source, in the target's
// basis e_a, e_b (et, ep), H_ab = (q/2pi) [delta_ab (1 - n.d)/|d|^2 - 2 (e_a.d)
// (e_b.d)/|d|^4]; the lane sums hd = sum q (1 - n.d)/|d|^2 and h_ab = sum q
// (e_a.d)(e_b.d)/|d|^4 (coincident points add nothing).
template <bool NPM>
__device__ __forceinline__ void tile_pairs_hess(const TileF32& t, const NpmK& nk, int r, int L, int tn, double ax, double ay, double az,
                                                const double* et, const double* ep, double* acc) {
    const float axh = (float)ax, ayh = (float)ay, azh = (float)az;
    const float axl = (float)(ax - (double)axh), ayl = (float)(ay - (double)ayh), azl = (float)(az - (double)azh);
    const float etf[3] = {(float)et[0], (float)et[1], (float)et[2]};
    const float epf[3] = {(float)ep[0], (float)ep[1], (float)ep[2]};
    constexpr float kLn2f = 0.693147180559945309f, kLog4f = 1.38629436111989061f;
    float f[8] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f}, c0 = 0.0f;
    for (int j = r; j < tn; j += L) {
        const float4 h = t.hi[j], l = t.lo[j];
        const float dx = (axh - h.x) + (axl - l.x);
        const float dy = (ayh - h.y) + (ayl - l.y);
        const float dz = (azh - h.z) + (azl - l.z);
        const float d2 = dx * dx + dy * dy + dz * dz;
        const bool coinc = d2 == 0.0f;
        const float r2 = coinc ? 1.0f : d2;
        float lg = coinc ? kLog4f : __builtin_amdgcn_logf(r2) * kLn2f;
        const float i0 = __builtin_amdgcn_rcpf(r2);
        float wi = h.w * i0;
        float wm = coinc ? 0.0f : wi;
        float w2 = wm * i0;
        if constexpr (NPM) {
            if (d2 < (float)nk.four_t) {
                const float u = 0.25f * d2, v = u * (float)nk.inv_t, omu = 1.0f - u;
                lg = npm_interior_log(v, (float)nk.t, (float)nk.ln4t, nk.nterms);
                wi = h.w * 0.25f * (2.0f * (float)nk.inv_t - v * (float)nk.inv_t - 1.0f) / omu;
                wm = wi;
                w2 = h.w * (float)nk.a2 / (omu * omu);
            }
        }
        const float y = fmaf(h.w, lg, -c0);  // Kahan-compensated log terms, as in tile_pairs
        const float tt = f[0] + y;
        c0 = (tt - f[0]) - y;
        f[0] = tt;
        f[1] = fmaf(wi, dx, f[1]);
        f[2] = fmaf(wi, dy, f[2]);
        f[3] = fmaf(wi, dz, f[3]);
        // 1 - n.d = 1 - |d|^2/2 for unit vectors (n.d = |d|^2 / 2)
        const float da = etf[0] * dx + etf[1] * dy + etf[2] * dz;
        const float db = epf[0] * dx + epf[1] * dy + epf[2] * dz;
        f[4] = fmaf(-0.5f * d2, wm, f[4] + wm);
        f[5] = fmaf(w2 * da, da, f[5]);
        f[6] = fmaf(w2 * da, db, f[6]);
        f[7] = fmaf(w2 * db, db, f[7]);
    }
    acc[0] += (double)f[0] - (double)c0;
#pragma unroll
    for (int k = 1; k < 8; ++k) acc[k] += (double)f[k];
}

// FP64 pair terms of TB targets of one lane over one LDS tile.  a[b]: the
// target; acc[b]: S, V (and, HESS, hd = sum q (1 - n.d)/|d|^2 and h_ab = sum q
// (e_a.d)(e_b.d)/|d|^4 in the target's basis e[b], Sec. 2.2: H_ab = (q/2pi)
// [delta_ab (1 - n.d)/|d|^2 - 2 (e_a.d)(e_b.d)/|d|^4]; coincident points add
// nothing).  Coincident points, |d|^2 = 0, take |d|^2 = 4 instead (log 4, and
// d = 0 zeroes their deflection): both have a zero low word, so only the high
// word is switched.  |d|^2 may be subnormal (two points beside a pole or an
// axis, 1e-155 apart).
struct TileF64 {
    double4 p[kTile];
};

__device__ __forceinline__ void tile_store(TileF64& t, int k, double4 v) { t.p[k] = v; }

template <int TB, bool HESS, bool NPM>
__device__ __forceinline__ void tile_pairs(const TileF64& t, const double2* ltab, const LogPoly& lk, const NpmK& nk,
                                           int r, int L, int tn, const double (*a)[3], const double (*e)[6],
                                           double (*acc)[HESS ? 8 : 4]) {
    if (r >= tn) return;
    double4 nx = t.p[r];
    for (int j = r; j < tn; j += L) {
        const double4 sp = nx;
        nx = t.p[min(j + L, kTile - 1)];  // the next particle, read ahead
        double d[TB][3], d2r[TB], m[TB];
        int ex[TB];
        double2 tab[TB];
#pragma unroll
        for (int b = 0; b < TB; ++b) {
            d[b][0] = a[b][0] - sp.x;
            d[b][1] = a[b][1] - sp.y;
            d[b][2] = a[b][2] - sp.z;
            d2r[b] = d[b][0] * d[b][0] + d[b][1] * d[b][1] + d[b][2] * d[b][2];
            m[b] = frexp(__hiloint2double(d2r[b] == 0.0 ? 0x40100000 : __double2hiint(d2r[b]), __double2loint(d2r[b])),
                         &ex[b]);
            tab[b] = log_tab_at((uint32_t)__double2hiint(m[b]), ltab);
        }
        __builtin_amdgcn_sched_barrier(0);  // every table read is under way before the first is waited for
#pragma unroll
        for (int b = 0; b < TB; ++b) {
            double lg, i0;
            log_recip_at(m[b], ex[b], tab[b], lk, &lg, &i0);
            double wi = sp.w * i0, wm = wi, w2 = 0.0;
            if constexpr (HESS) {
                wm = d2r[b] == 0.0 ? 0.0 : wi;
                w2 = wm * i0;
            }
            if constexpr (NPM) {
                if (d2r[b] < nk.four_t) {
                    const double u = 0.25 * d2r[b], v = u * nk.inv_t, omu = 1.0 - u;
                    lg = npm_interior_log(v, nk.t, nk.ln4t, nk.nterms);
                    wi = sp.w * 0.25 * (2.0 * nk.inv_t - v * nk.inv_t - 1.0) / omu;
                    wm = wi;
                    w2 = sp.w * nk.a2 / (omu * omu);
                }
            }
            acc[b][0] = fma(sp.w, lg, acc[b][0]);
            acc[b][1] = fma(wi, d[b][0], acc[b][1]);
            acc[b][2] = fma(wi, d[b][1], acc[b][2]);
            acc[b][3] = fma(wi, d[b][2], acc[b][3]);
            if constexpr (HESS) {
                const double nd = a[b][0] * d[b][0] + a[b][1] * d[b][1] + a[b][2] * d[b][2];
                const double da = e[b][0] * d[b][0] + e[b][1] * d[b][1] + e[b][2] * d[b][2];
                const double db = e[b][3] * d[b][0] + e[b][4] * d[b][1] + e[b][5] * d[b][2];
                acc[b][4] = fma(-nd, wm, acc[b][4] + wm);
                acc[b][5] = fma(w2 * da, da, acc[b][5]);
                acc[b][6] = fma(w2 * da, db, acc[b][6]);
                acc[b][7] = fma(w2 * db, db, acc[b][7]);
            }
        }
    }
}

// Workgroups of four waves that share the log table.  WPI = 1: every wave
// takes an item of its own, with no barrier after the table's (items are
// sorted by work, so the four are alike).  WPI = 4
// (few items, kP2PFewItems): the workgroup takes one item, every wave decodes
// its entries by itself and takes every fourth tile, and the sums are added
// over the waves; 228 leaves of 80,000 pairs each took 325 us as one wave
// each, 61 us so.  Where there are many items the waves' repeated decoding
// costs more than it gives (clustered-1e7: 3.1 ms).
//   FP64: a lane takes TB = 2 targets against each particle it reads, so the
//   LDS return path (3 x 16 bytes a pair for the particle and the table entry,
//   128 bytes a cycle) stays behind the VALU, and ng targets keep
//   2 floor(64 / ceil(ng / 2)) lanes busy where teams of floor(64 / ng) left
//   up to half of them idle.  Where the leaves have kP2POneTarget targets each
//   or fewer on average, an item is too short for that: its tiles' latency
//   counts, one target a lane leaves room for a fifth wave per SIMD, and a
//   grid of kP2POneGrid workgroups makes the table fewer times (us, two
//   targets without and one with the bounded grid: 1e6 targets in 223,000
//   leaves 637 and 506; 2e6 in 708,000 leaves 2,216 and 1,703; 2e5 in 126,000
//   leaves of a clustered sky 523 and 394).  Two targets win from some 9 a
//   leaf (10.2: 1,634 against 1,717 us; 8.5: 718 against 661), and gain
//   nothing from the bounded grid (868 and 905 us).
//   FP32 (precision tier): a target per lane and teams of floor(64 / ng), as
//   the order of its FP32 tile sums is part of its result.
constexpr int kP2PFewItems = 4096;
constexpr int64_t kP2POneTarget = 8;
constexpr unsigned kP2POneGrid = 4096;
// waves of a workgroup: the precision tier needs no table, so its one-wave
// items go one to a workgroup (nothing waits for the longest of four)
constexpr int p2p_waves(bool f32, int wpi) { return wpi > 1 ? wpi : f32 ? 1 : 4; }

template <int WPI>
__device__ __forceinline__ void team_sync() {
    if constexpr (WPI > 1) {
        __syncthreads();
    } else {  // one wave: its LDS operations stay in order
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
}

constexpr int p2p_waves_per_simd(bool f32, bool wide, int tb) { return wide ? 2 : f32 ? 6 : tb == 1 ? 5 : 4; }

template <bool F32, bool HESS, bool NPM, int WPI, int TB>
__global__ void __launch_bounds__(64 * p2p_waves(F32, WPI))
    __attribute__((amdgpu_waves_per_eu(p2p_waves_per_simd(F32, HESS || NPM, TB))))
k_p2p(FmmCtx c, const int4* __restrict__ items, int nitems, const int* __restrict__ src,
      const int* __restrict__ tfirst, const int* __restrict__ tcount, const double* __restrict__ tx,
      const double* __restrict__ ty, const double* __restrict__ tz, double* __restrict__ near, int64_t m,
      double* __restrict__ part, LogPoly lk, double* __restrict__ hess, NpmK nk) {
    using Tile = std::conditional_t<F32, TileF32, TileF64>;
    constexpr int NR = HESS ? 8 : 4, NT = 64 * WPI, kP2PWaves = p2p_waves(F32, WPI);
    // a wave's tile and its part of the end-of-group reduction share LDS
    static_assert(sizeof(Tile) >= NR * 64 * sizeof(double), "the reduction fits the tile");
    __shared__ __align__(16) unsigned char sm[sizeof(Tile) * kP2PWaves];
    __shared__ double fin[kP2PWaves / WPI][NR][64];
    __shared__ double2 ltab[F32 ? 1 : kLogTab];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int wave = WPI > 1 ? wv : 0, tid = WPI > 1 ? threadIdx.x : lane;  // within the item's team
    const int team = WPI > 1 ? 0 : wv;
    Tile& tile = reinterpret_cast<Tile*>(sm)[wv];
    double(*red)[64] = reinterpret_cast<double(*)[64]>(sm + sizeof(Tile) * (WPI > 1 ? 0 : wv));  // [wave NR + q]
    constexpr int RW = sizeof(Tile) / (64 * sizeof(double));  // rows of one wave's part
    if constexpr (!F32) {
        for (int j = threadIdx.x; j < kLogTab; j += 64 * kP2PWaves) ltab[j] = log_tab_entry(j);
    }
    if (kP2PWaves > 1) __syncthreads();
    // one coefficient in a vector register: an FMA reads one scalar operand
    asm("" : "+v"(lk.c4));
    const int ew = 2 * c.p + 2;
    const double4* __restrict__ spt = c.spt;
    // uniform across the item's team (WPI > 1: one item a workgroup); nitems is
    // an int, so the last step stays below 2^32
    constexpr bool kStrided = !F32 && TB == 1;  // the others' grids hold every item
    for (unsigned it = WPI > 1 ? blockIdx.x : blockIdx.x * kP2PWaves + wv; it < (unsigned)nitems;
         it = kStrided ? it + gridDim.x * kP2PWaves : ~0u) {
        const int4 item = items[it];
        const int T = item.x;
        const int k0 = item.y, K = item.z - item.y;
        const int t0 = tfirst[T], nt = tcount[T];
        for (int tg = 64 * blockIdx.y; tg < nt; tg += 64 * gridDim.y) {
            const int ng = min(64, nt - tg);
            const int g0 = t0 + tg;
            const int nb = (ng + TB - 1) / TB;  // blocks of TB targets
            const int L = 64 / nb;              // lanes per block
            const int blk = lane / L, r = lane - blk * L;
            const bool active = blk < nb;
            double a[TB][3], e[TB][6], acc[TB][NR];
#pragma unroll
            for (int b = 0; b < TB; ++b) {
                const int my = g0 + (active ? min(blk * TB + b, ng - 1) : 0);
                a[b][0] = tx[my];
                a[b][1] = ty[my];
                a[b][2] = tz[my];
                if constexpr (HESS) target_basis(a[b][0], a[b][1], a[b][2], e[b], e[b] + 3);
#pragma unroll
                for (int q = 0; q < NR; ++q) acc[b][q] = 0.0;
            }
            double qnear = 0.0;  // lane partials of Q_near (every wave of a team has them all)
            for (int kc = 0; kc < K; kc += 64) {
                const int kk = min(64, K - kc);
                int cnt = 0, fst = 0;
                if (lane < kk) {
                    const int S = src[k0 + kc + lane];
                    cnt = c.count[S];
                    fst = c.first[S];
                    qnear += c.mult[(size_t)S * ew + 1] * (4.0 * M_PI);
                }
                // inclusive wave scan of the counts
                int incl = cnt;
#pragma unroll
                for (int o = 1; o < 64; o <<= 1) {
                    const int v = __shfl_up(incl, o, 64);
                    if (lane >= o) incl += v;
                }
                const int excl = (lane < kk) ? incl - cnt : 0x7fffffff;
                const int total = __shfl(incl, 63, 64);
                for (int s0 = wave * kTile; s0 < total; s0 += WPI * kTile) {
                    const int tn = min(kTile, total - s0);
                    double4 v[kTile / 64];
#pragma unroll
                    for (int j = 0; j < kTile / 64; ++j) {
                        const int f = s0 + j * 64 + lane;
                        // entry e: the last one whose start is <= f
                        int e_ = 0;
#pragma unroll
                        for (int step = 32; step > 0; step >>= 1) {
                            const int cand = e_ + step;
                            if (__shfl(excl, cand, 64) <= f) e_ = cand;
                        }
                        const int base = __shfl(fst, e_, 64) - __shfl(excl, e_, 64);
                        v[j] = spt[base + min(f, total - 1)];  // past the end: the last particle again
                    }
                    team_sync<1>();  // the wave's last tile is consumed
#pragma unroll
                    for (int j = 0; j < kTile / 64; ++j) tile_store(tile, j * 64 + lane, v[j]);
                    team_sync<1>();
                    if (active) {
                        if constexpr (!F32) tile_pairs<TB, HESS, NPM>(tile, ltab, lk, nk, r, L, tn, a, e, acc);
                        else if constexpr (HESS)
                            tile_pairs_hess<NPM>(tile, nk, r, L, tn, a[0][0], a[0][1], a[0][2], e[0], e[0] + 3,
                                                 acc[0]);
                        else
                            tile_pairs<NPM>(tile, nk, r, L, tn, a[0][0], a[0][1], a[0][2], acc[0][0], acc[0][1],
                                            acc[0][2], acc[0][3]);
                    }
                }
            }
            const double qn = wave_sum(qnear);
#pragma unroll
            for (int b = 0; b < TB; ++b) {
                team_sync<WPI>();  // the tiles (or the other target's sums) are consumed
#pragma unroll
                for (int q = 0; q < NR; ++q) red[wave * RW + q][lane] = acc[b][q];
                team_sync<WPI>();
                for (int x = tid; x < nb * NR; x += NT) {
                    const int q = x / nb, k = x - q * nb;
                    if (k * TB + b >= ng) continue;
                    double s = 0.0;
                    for (int w = 0; w < WPI; ++w)
                        for (int l = 0; l < L; ++l) s += red[w * RW + q][k * L + l];
                    fin[team][q][k * TB + b] = s;
                }
            }
            team_sync<WPI>();
            if (tid < ng) {
                const double(*fs)[64] = fin[team];
                const int me = g0 + tid;
                const double s0 = fs[0][tid], s1 = fs[1][tid], s2 = fs[2][tid], s3 = fs[3][tid];
                const double mx = tx[me], myy = ty[me], mz = tz[me];
                const double il = 1.0 / sqrt(mx * mx + myy * myy + mz * mz);
                const double ux = mx * il, uy = myy * il, uz = mz * il;
                const double vr = ux * s1 + uy * s2 + uz * s3;
                const int slot = item.w < 0 ? -1 : item.w + tg + tid;
                if constexpr (HESS) {
                    const double h4 = fs[4][tid], h5 = fs[5][tid], h6 = fs[6][tid], h7 = fs[7][tid];
                    const double h[3] = {(h4 - 2.0 * h5) * kInv2Pi, -2.0 * h6 * kInv2Pi, (h4 - 2.0 * h7) * kInv2Pi};
                    emit_target_hess(slot, me, (s0 + (1.0 - kLog4) * qn) * kInv4Pi, (s1 - ux * vr) * kInv2Pi,
                                     (s2 - uy * vr) * kInv2Pi, (s3 - uz * vr) * kInv2Pi, h, part, near, hess, m);
                } else {
                    emit_target(slot, me, (s0 + (1.0 - kLog4) * qn) * kInv4Pi, (s1 - ux * vr) * kInv2Pi,
                                (s2 - uy * vr) * kInv2Pi, (s3 - uz * vr) * kInv2Pi, part, near, m);
                }
            }
            team_sync<WPI>();  // fin and the tiles are reused by the next group
        }
    }
}

// ------------------------------------------------------------ multipole evaluations
// One 64-wide workgroup per target leaf with far entries, targets in groups
// of ng <= 64 and lanes in teams of L = floor(64 / ng) as in k_p2p.  The far
// leaves are taken kChunkF at a time: their expansion records and frames
// are loaded once into LDS (coalesced: each record is contiguous), then
// lane r of team t evaluates leaves r, r + L, ... of the chunk at target t.
// The team's partial sums are added in a fixed order at the end of the
// group.
constexpr int kChunkF = 16;

template <int P, bool HESS>
__global__ void __launch_bounds__(64) k_m2p(FmmCtx c, const int4* __restrict__ items,
                                           const int* __restrict__ src, const int* __restrict__ tfirst,
                                           const int* __restrict__ tcount, const double* __restrict__ tx,
                                           const double* __restrict__ ty, const double* __restrict__ tz,
                                           double* __restrict__ near, int64_t m, double* __restrict__ part,
                                           double* __restrict__ hess) {
    constexpr int EW = 2 * P + 2;
    // the staged records double as the end-of-group reduction buffer
    static_assert(kChunkF * (2 * kM2PMinOrder + 2) >= 4 * 64, "reduction fits the record buffer");
    __shared__ __align__(16) double coef[kChunkF * EW];
    __shared__ double frm[kChunkF][10];  // c, e_theta, e_phi, rho
    double(*red)[64] = reinterpret_cast<double(*)[64]>(coef);
    __shared__ double redh[HESS ? 3 : 1][64];  // the Hessian's partials
    const int lane = threadIdx.x;
    const int4 item = items[blockIdx.x];
    const int T = item.x;
    const int k0 = item.y, K = item.z - item.y;
    const int t0 = tfirst[T], nt = tcount[T];
    for (int tg = 64 * blockIdx.y; tg < nt; tg += 64 * gridDim.y) {
        const int ng = min(64, nt - tg);
        const int g0 = t0 + tg;
        const int L = 64 / ng;
        const int team = lane / L, r = lane - team * L;
        const bool active = team < ng;
        const int my = g0 + (active ? team : 0);
        const double nx = tx[my], ny = ty[my], nz = tz[my];
        double p0 = 0.0, p1 = 0.0, p2 = 0.0, p3 = 0.0;
        double hs[3] = {0.0, 0.0, 0.0};
        double et[3], ep[3];
        if constexpr (HESS) target_basis(nx, ny, nz, et, ep);
        for (int kc = 0; kc < K; kc += kChunkF) {
            const int cf = min(kChunkF, K - kc);
            __syncthreads();  // previous chunk fully consumed
            // records are EW = 2P + 2 doubles (16-byte aligned): copied as
            // double2, P + 1 per record
#pragma unroll 4
            for (int idx = lane; idx < cf * (P + 1); idx += 64) {
                const int f = idx / (P + 1), e = idx - f * (P + 1);
                reinterpret_cast<double2*>(coef)[idx] =
                    reinterpret_cast<const double2*>(c.mult + (size_t)src[k0 + kc + f] * EW)[e];
            }
            if (lane < cf) {
                const double* cs = c.cen + 4 * (size_t)src[k0 + kc + lane];
                const Frame fr = make_frame(cs[0], cs[1], cs[2]);
#pragma unroll
                for (int d = 0; d < 3; ++d) {
                    frm[lane][d] = fr.c[d];
                    frm[lane][3 + d] = fr.et[d];
                    frm[lane][6 + d] = fr.ep[d];
                }
                frm[lane][9] = cs[3];
            }
            __syncthreads();
            if (active) {
                for (int j = r; j < cf; j += L) {
                    Frame fr;
#pragma unroll
                    for (int d = 0; d < 3; ++d) {
                        fr.c[d] = frm[j][d];
                        fr.et[d] = frm[j][3 + d];
                        fr.ep[d] = frm[j][6 + d];
                    }
                    double ps, ax, ay, az;
                    if constexpr (HESS) {
                        double h[3];
                        m2p_eval_hess<P>(coef + j * EW, fr, frm[j][9], nx, ny, nz, et, ep, &ps, &ax, &ay, &az, h);
                        hs[0] += h[0];
                        hs[1] += h[1];
                        hs[2] += h[2];
                    } else {
                        m2p_eval<P>(coef + j * EW, fr, frm[j][9], nx, ny, nz, &ps, &ax, &ay, &az);
                    }
                    p0 += ps;
                    p1 += ax;
                    p2 += ay;
                    p3 += az;
                }
            }
        }
        __syncthreads();  // the last chunk fully consumed before red overwrites it
        red[0][lane] = p0;
        red[1][lane] = p1;
        red[2][lane] = p2;
        red[3][lane] = p3;
        if constexpr (HESS) {
            redh[0][lane] = hs[0];
            redh[1][lane] = hs[1];
            redh[2][lane] = hs[2];
        }
        __syncthreads();
        if (lane < ng) {
            double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
            double h[3] = {0.0, 0.0, 0.0};
            for (int j = lane * L; j < lane * L + L; ++j) {
                s0 += red[0][j];
                s1 += red[1][j];
                s2 += red[2][j];
                s3 += red[3][j];
                if constexpr (HESS) {
                    h[0] += redh[0][j];
                    h[1] += redh[1][j];
                    h[2] += redh[2][j];
                }
            }
            if constexpr (HESS)
                emit_target_hess(item.w < 0 ? -1 : item.w + tg + lane, g0 + lane, s0, s1, s2, s3, h, part,
                                 near, hess, m);
            else
                emit_target(item.w < 0 ? -1 : item.w + tg + lane, g0 + lane, s0, s1, s2, s3, part, near, m);
        }
        __syncthreads();  // red is reused by the next group
    }
}

void reduce_items(const WorkItems& w, const int* tfirst, const int* tcount, double* near, int64_t m, double* part,
                  hipStream_t s, double* hess) {
    if (w.nred <= 0) return;
    const dim3 g((unsigned)w.nred, target_groups(m, w.nred));
    if (hess) k_near_reduce<true><<<g, 64, 0, s>>>(w.red, tfirst, tcount, part, near, hess, m);
    else k_near_reduce<false><<<g, 64, 0, s>>>(w.red, tfirst, tcount, part, near, nullptr, m);
    SFMM_LAUNCH_CHECK();
}

void fmm_p2p(const FmmCtx& c, bool fp32, const WorkItems& w, const int* src, const int* tfirst,
             const int* tcount, const double* tx, const double* ty, const double* tz, double* near, int64_t m,
             hipStream_t s, double* part, double* hess) {
    if (w.n <= 0) return;
    if (hess && !part && w.nred > 0) throw Error(ST_INTERNAL, "the Hessian needs partial slots of 8 doubles");
    if (!part) part = w.part;
    const NpmK nk = npm_params(c.npm_sigma);
    const bool npm = c.npm_sigma > 0.0;
    // few items: a workgroup each, groups of 64 targets of one leaf side by side
    const bool few = w.n < kP2PFewItems;
    const int pw = p2p_waves(fp32, few ? 4 : 1);
    // leaves with few targets: one target a lane, a bounded grid
    const bool one = !fp32 && !few && !hess && !npm && m <= kP2POneTarget * (int64_t)w.leaves;
    const unsigned gx = few ? (unsigned)w.n : one ? std::min(nblk(w.n, pw), kP2POneGrid) : nblk(w.n, pw);
    const dim3 g(gx, std::max(few ? 2u : 1u, target_groups(m, w.n)));
#define P2P_W(T, H, N, W, B)                                                                                   \
    k_p2p<T, H, N, W, B><<<g, 64 * pw, 0, s>>>(c, w.items, w.n, src, tfirst, tcount, tx, ty, tz, near, m, part, \
                                               kLogPoly, hess, nk)
#define P2P_(T, H, N)                        \
    if (few) P2P_W(T, H, N, 4, (T ? 1 : 2)); \
    else P2P_W(T, H, N, 1, (T ? 1 : 2))
#define P2P_N(T, H)                  \
    if (npm) {                       \
        P2P_(T, H, true);            \
    } else {                         \
        P2P_(T, H, false);           \
    }
    if (one) {
        P2P_W(false, false, false, 1, 1);
    } else if (fp32) {
        if (hess) P2P_N(true, true) else P2P_N(true, false)
    } else {
        if (hess) P2P_N(false, true) else P2P_N(false, false)
    }
#undef P2P_N
#undef P2P_
#undef P2P_W
    SFMM_LAUNCH_CHECK();
    reduce_items(w, tfirst, tcount, near, m, part, s, hess);
}

void fmm_m2p(const FmmCtx& c, const WorkItems& w, const int* src, const int* tfirst, const int* tcount,
             const double* tx, const double* ty, const double* tz, double* near, int64_t m, hipStream_t s,
             double* part, double* hess) {
    if (w.n <= 0 || c.p < kM2PMinOrder) return;
    if (hess && !part && w.nred > 0) throw Error(ST_INTERNAL, "the Hessian needs partial slots of 8 doubles");
    if (!part) part = w.part;
    const dim3 g((unsigned)w.n, target_groups(m, w.n));
#define L_(P)                                                                                                \
    case P:                                                                                                  \
        if (hess) k_m2p<P, true><<<g, 64, 0, s>>>(c, w.items, src, tfirst, tcount, tx, ty, tz, near, m, part, \
                                                  hess);                                                     \
        else k_m2p<P, false><<<g, 64, 0, s>>>(c, w.items, src, tfirst, tcount, tx, ty, tz, near, m, part,    \
                                              nullptr);                                                      \
        break;
    SFMM_DISPATCH(c.p, L_)
#undef L_
    SFMM_LAUNCH_CHECK();
    reduce_items(w, tfirst, tcount, near, m, part, s, hess);
}

double npm_constant(double sigma) {
    if (!(sigma > 0.0)) return 0.0;
    const double st = std::sin(0.5 * sigma), t = st * st;
    double J = 0.0, tk = 1.0;
    for (int k = 0; k < 200 && tk > 1e-18; ++k, tk *= t) J += tk * ((2.0 - t) / (k + 2) - 1.0 / (k + 3));
    return t * (J - 1.0);
}

NpmK npm_params(double sigma) {
    NpmK k{};
    if (!(sigma > 0.0)) return k;
    const double st = std::sin(0.5 * sigma);
    k.t = st * st;
    k.inv_t = 1.0 / k.t;
    k.four_t = 4.0 * k.t;
    k.ln4t = std::log(4.0 * k.t);
    const double a = (1.0 - k.t) / k.t;
    k.a2 = a * a / 16.0;
    // terms of the series for I until t^k < 2^-56 (v <= 1)
    k.nterms = 1;
    for (double tk = k.t; tk >= 0x1p-56 && k.nterms < 64; tk *= k.t) ++k.nterms;
    return k;
}

}  // namespace sfmm

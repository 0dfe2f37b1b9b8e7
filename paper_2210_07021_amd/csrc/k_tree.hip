// Tree build on the GPU: order-29 HEALPix keys (Sec. 3.1), the adaptive
// quasi-quad-tree from the common prefixes of the sorted keys, all levels at
// once, target location (Sec. 3.7), and the frontier form of Algorithm 1 (Sec.
// 3.4) that makes the full lists of the exports and statistics.
#include "common.hpp"
#include "geom.hpp"

#include <algorithm>

namespace sfmm {

static unsigned nblocks(int64_t n, int b) { return (unsigned)((n + b - 1) / b > 0 ? (n + b - 1) / b : 1); }

// ------------------------------------------------------------------ points
// Unit vectors, keys and identity permutation of n points given as [3][n];
// each point is written as one 32-byte record (x, y, z, q) so that the
// gather after the key sort moves one aligned record per point (q = 0 when
// the points carry no charge).
__global__ void k_prepare_points(const double* in, const double* q, int64_t n, double4* u, uint64_t* keys,
                                 uint32_t* idx, volatile int* err) {
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= n) return;
    double a = in[i], b = in[n + i], c = in[2 * n + i];
    const double r2 = a * a + b * b + c * c;
    int e = 0;
    if (!(isfinite(a) && isfinite(b) && isfinite(c))) e |= 1;
    else if (!(fabs(r2 - 1.0) <= 2e-6)) e |= 2;
    if (e) {
        err[e - 1] = 1;  // host memory, one int per kind
        a = 0.0; b = 0.0; c = 1.0;
    } else if (fabs(r2 - 1.0) > 1e-14) {
        const double inv = 1.0 / sqrt(r2);
        a *= inv; b *= inv; c *= inv;
    }
    u[i] = make_double4(a, b, c, q ? q[i] : 0.0);
    keys[i] = key29(a, b, c);
    idx[i] = (uint32_t)i;
}

void prepare_points(const double* in, const double* q, int64_t n, double4* u, uint64_t* keys, uint32_t* idx,
                    int* err, hipStream_t s) {
    if (n <= 0) return;
    k_prepare_points<<<nblocks(n, 256), 256, 0, s>>>(in, q, n, u, keys, idx, err);
    SFMM_LAUNCH_CHECK();
}

// Targets in plan order: coordinates (SoA) and leaf box of the target at
// each position, from the leaf-sorted (leaf, index) pairs.
__global__ void k_gather_targets(const uint32_t* idx, const uint64_t* leaf_sorted, int64_t n,
                                 const double4* __restrict__ u, double* ox, double* oy, double* oz, int* leaf) {
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= n) return;
    const double4 v = u[idx[i]];
    ox[i] = v.x;
    oy[i] = v.y;
    oz[i] = v.z;
    leaf[i] = (int)leaf_sorted[i];
}

void gather_targets(const uint32_t* idx, const uint64_t* leaf_sorted, int64_t n, const double4* u, double* ox,
                    double* oy, double* oz, int* leaf, hipStream_t s) {
    if (n <= 0) return;
    k_gather_targets<<<nblocks(n, 256), 256, 0, s>>>(idx, leaf_sorted, n, u, ox, oy, oz, leaf);
    SFMM_LAUNCH_CHECK();
}

__global__ void k_gather_records(const uint32_t* idx, int64_t n, const double4* __restrict__ u, double4* out) {
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i < n) out[i] = u[idx[i]];
}

void gather_records(const uint32_t* idx, int64_t n, const double4* u, double4* out, hipStream_t s) {
    if (n <= 0) return;
    k_gather_records<<<nblocks(n, 256), 256, 0, s>>>(idx, n, u, out);
    SFMM_LAUNCH_CHECK();
}

// ------------------------------------------------------------------ tree
// The whole tree at once from the sorted keys.  A box of level L holds more
// than m points exactly when its first point i and point i + m share its
// pixel, and i is the first point of its level-L pixel exactly when point i -
// 1 does not share it.  So with common(i, j) the deepest level at which keys i
// and j share a pixel, the split boxes that start at point i are those of the
// levels common(i - 1, i) < L <= min(common(i, i + m), max_level - 1).  One
// pass counts them per level, a scan gives every split box its place in its
// level's list (ordered by first point), one pass writes their first points,
// and a last one cuts every split box's points into its four children: split
// s has the children 12 + 4s .. 12 + 4s + 3.  Against two launches a level and
// a read-back every eight levels (24 levels: 0.40 ms of kernels on
// clustered-1e7, and most of a small plan's tree time is launches) the passes
// read the keys twice.
__device__ int lower_bound_u64(const uint64_t* a, int lo, int hi, uint64_t v) {
    while (lo < hi) {
        const int mid = lo + ((hi - lo) >> 1);
        if (a[mid] < v) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

// first index in [lo, hi) of a sorted int list with a[] >= v
__device__ __forceinline__ int lower_bound_i32(const int* a, int lo, int hi, int v) {
    while (lo < hi) {
        const int mid = lo + ((hi - lo) >> 1);
        if (a[mid] < v) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

// deepest level at which two order-29 keys share a pixel (-1: none)
__device__ __forceinline__ int common_level(uint64_t a, uint64_t b) {
    const uint64_t x = a ^ b;
    return x == 0 ? kOrder : max(-1, kOrder - 1 - (63 - (int)__clzll((long long)x)) / 2);
}

// Bits of the levels of the split boxes that start at point i.
__device__ __forceinline__ uint32_t split_levels(const uint64_t* __restrict__ keys, int64_t n, int64_t i, int64_t m,
                                                 int max_level) {
    if (i + m >= n) return 0;
    const uint64_t k = keys[i];
    const int c = min(common_level(k, keys[i + m]), max_level - 1);
    const int d = i == 0 ? -1 : common_level(keys[i - 1], k);
    return c > d ? (uint32_t)((2ull << c) - (1ull << (d + 1))) : 0u;
}

// A wave takes kMarkPoints consecutive points, 64 at a time; lane L holds the
// running count of level L.  EMIT: it starts from the scanned counts, and
// every split box's first point goes to its place.
constexpr int kMarkPoints = 512;
template <bool EMIT>
__global__ void __launch_bounds__(256) k_tree_mark(const uint64_t* __restrict__ keys, int64_t n, int64_t m,
                                                   int max_level, int nt, int* __restrict__ cnt,
                                                   TreeLevels lv, int* __restrict__ sfirst) {
    const int tile = (int)((blockIdx.x * (int64_t)blockDim.x + threadIdx.x) >> 6), lane = threadIdx.x & 63;
    if (tile >= nt) return;  // uniform across the wave
    const uint64_t lt = (1ull << lane) - 1;
    int run = EMIT && lane < kTreeLevels ? cnt[(size_t)lane * nt + tile] + lv.soff[lane] : 0;
    for (int k = 0; k < kMarkPoints; k += 64) {
        const int64_t i = (int64_t)tile * kMarkPoints + k + lane;
        const uint32_t bits = split_levels(keys, n, i, m, max_level);
        uint32_t any = bits;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) any |= __shfl_xor(any, o, 64);
        any = __builtin_amdgcn_readfirstlane(any);
        while (any) {
            const int L = __ffs(any) - 1;
            any &= any - 1;
            const uint64_t mask = __ballot(bits >> L & 1);
            if (EMIT) {
                const int base = __builtin_amdgcn_readlane(run, L);
                if (bits >> L & 1) sfirst[base + __popcll(mask & lt)] = (int)i;
            }
            if (lane == L) run += __popcll(mask);
        }
    }
    if (!EMIT && lane < kTreeLevels) cnt[(size_t)lane * nt + tile] = run;
}

int tree_tiles(int64_t n) { return (int)std::max<int64_t>(1, (n + kMarkPoints - 1) / kMarkPoints); }

void tree_count(const uint64_t* keys, int64_t n, int m, int max_level, int* cnt, hipStream_t s) {
    const int nt = tree_tiles(n);
    k_tree_mark<false><<<nblocks((int64_t)nt * 64, 256), 256, 0, s>>>(keys, n, m, max_level, nt, cnt, TreeLevels{},
                                                                      nullptr);
    SFMM_LAUNCH_CHECK();
}

void tree_emit(const uint64_t* keys, int64_t n, int m, int max_level, int* cnt, const TreeLevels& lv, int* sfirst,
               hipStream_t s) {
    const int nt = tree_tiles(n);
    k_tree_mark<true><<<nblocks((int64_t)nt * 64, 256), 256, 0, s>>>(keys, n, m, max_level, nt, cnt, lv, sfirst);
    SFMM_LAUNCH_CHECK();
}

// Four lanes per split box: lane q finds where child q ends (from the box's
// first point in growing steps, then by bisection), writes the child, and
// looks up the child's own split (child0) and the box's index (the children's
// parent) in the level lists.  The first workgroup's first 12 threads write
// the base pixels instead.  Bound by the chain of dependent loads (~40, a few
// of them past the L2).
__global__ void __launch_bounds__(256) k_tree_boxes(const uint64_t* __restrict__ keys, int n, int m, int max_level,
                                                    TreeLevels lv, const int* __restrict__ sfirst, int nsplit,
                                                    int* __restrict__ level, uint64_t* __restrict__ pixel,
                                                    int* __restrict__ first, int* __restrict__ count,
                                                    int* __restrict__ parent, int* __restrict__ child0) {
    if (blockIdx.x == 0) {
        const int f = threadIdx.x;
        if (f >= 12) return;
        const int a = lower_bound_u64(keys, 0, n, (uint64_t)f << (2 * kOrder));
        const int b = lower_bound_u64(keys, 0, n, (uint64_t)(f + 1) << (2 * kOrder));
        level[f] = 0;
        pixel[f] = (uint64_t)f;
        first[f] = a;
        count[f] = b - a;
        parent[f] = -1;
        child0[f] = b - a > m && max_level > 0 ? 12 + 4 * lower_bound_i32(sfirst, lv.soff[0], lv.soff[1], a) : -1;
        return;
    }
    const int t = (blockIdx.x - 1) * 256 + threadIdx.x;
    const int s = t >> 2, q = t & 3;
    if (s >= nsplit) return;  // the four lanes of a box leave together
    int L = 0;
    while (s >= lv.soff[L + 1]) ++L;
    const int i0 = sfirst[s];
    const uint64_t pix = keys[i0] >> (2 * (kOrder - L)), cp = 4 * pix + (uint64_t)q;
    const uint64_t v = (cp + 1) << (2 * (kOrder - L - 1));
    // the end of child q: keys[lo] < v (or lo = i0), keys[hi] >= v or hi = n
    int lo = i0, hi = n;
    for (int64_t step = 64; (int64_t)lo + step < n; step <<= 2) {
        if (keys[lo + step] < v) {
            lo += (int)step;
        } else {
            hi = lo + (int)step;
            break;
        }
    }
    const int end = lower_bound_u64(keys, lo, hi, v);
    const int st = __shfl_up(end, 1, 4);
    const int beg = q == 0 ? i0 : st;
    int b = (int)pix;
    if (L > 0) b = 12 + 4 * (lower_bound_i32(sfirst, lv.soff[L - 1], lv.soff[L], i0 + 1) - 1) + (int)(pix & 3);
    const int c = 12 + 4 * s + q;
    level[c] = L + 1;
    pixel[c] = cp;
    first[c] = beg;
    count[c] = end - beg;
    parent[c] = b;
    child0[c] = end - beg > m && L + 1 < max_level
                    ? 12 + 4 * lower_bound_i32(sfirst, lv.soff[L + 1], lv.soff[L + 2], beg)
                    : -1;
}

void tree_boxes(const uint64_t* keys, int64_t n, int m, int max_level, const TreeLevels& lv, const int* sfirst,
                int nsplit, int* level, uint64_t* pixel, int* first, int* count, int* parent, int* child0,
                hipStream_t s) {
    k_tree_boxes<<<1 + (nsplit > 0 ? nblocks(4 * (int64_t)nsplit, 256) : 0), 256, 0, s>>>(
        keys, (int)n, m, max_level, lv, sfirst, nsplit, level, pixel, first, count, parent, child0);
    SFMM_LAUNCH_CHECK();
}

// ------------------------------------------------------------------ walk records
__global__ void k_walk_boxes(int nb, const double* cen, const double* rad, const double* gdd, const int* child0,
                             const int* count, double c_s, double c_t, double sigma, double4* geo, double2* strig,
                             double4* ttrig, int2* cc, double* dtrig) {
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= nb) return;
    const double r = rad[b];
    geo[b] = make_double4(cen[4 * b], cen[4 * b + 1], cen[4 * b + 2], r);
    double s1, c1, s2, c2, s3, c3;
    sincos(protected_radius(r, c_s, sigma), &s1, &c1);
    sincos(r, &s2, &c2);
    sincos(r / c_t, &s3, &c3);
    strig[b] = make_double2(c1, s1);
    ttrig[b] = make_double4(c2, s2, c3, s3);
    cc[b] = make_int2(child0[b], count[b]);
    // double-double tables for the exact decisions of near-ties
    const dd R = {gdd[8 * (size_t)b + 6], gdd[8 * (size_t)b + 7]};
    const bool widen = sigma > 0.0 && r + sigma > c_s * r;
    const dd prot = widen ? dd_add(R, dd_from(sigma)) : dd_mul_d(R, c_s);
    const dd ang[3] = {prot, R, dd_div(R, dd_from(c_t))};
    double* o = dtrig + kWalkDtrig * (size_t)b;
    o[12] = prot.hi;
    o[13] = prot.lo;
    for (int k = 0; k < 3; ++k) {
        dd sn, cs;
        dd_sincos(ang[k], &sn, &cs);
        o[4 * k + 0] = cs.hi;
        o[4 * k + 1] = cs.lo;
        o[4 * k + 2] = sn.hi;
        o[4 * k + 3] = sn.lo;
    }
}

void walk_boxes(int nb, const double* cen, const double* rad, const double* gdd, const int* child0, const int* count,
                double c_s, double c_t, double sigma, double4* geo, double2* strig, double4* ttrig, int2* cc,
                double* dtrig, hipStream_t s) {
    if (nb <= 0) return;
    k_walk_boxes<<<nblocks(nb, 128), 128, 0, s>>>(nb, cen, rad, gdd, child0, count, c_s, c_t, sigma, geo, strig, ttrig,
                                                  cc, dtrig);
    SFMM_LAUNCH_CHECK();
}

// ------------------------------------------------------------------ targets
// Leaf box of each target from its key (any order of the targets), as the
// 64-bit sort key of the target order.
__global__ void k_locate(const uint64_t* keys, int64_t m, const int* child0, const int* level, uint64_t* leaf) {
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= m) return;
    const uint64_t k = keys[i];
    int b = (int)(k >> (2 * kOrder));
    while (child0[b] >= 0) {
        const int L = level[b] + 1;
        b = child0[b] + (int)((k >> (2 * (kOrder - L))) & 3);
    }
    leaf[i] = (uint64_t)b;
}

void locate_targets(const uint64_t* keys, int64_t m, const int* child0, const int* level, uint64_t* leaf,
                    hipStream_t s) {
    if (m <= 0) return;
    k_locate<<<nblocks(m, 256), 256, 0, s>>>(keys, m, child0, level, leaf);
    SFMM_LAUNCH_CHECK();
}

// Targets in plan order: each leaf's targets form one run.  The run's first
// target writes tfirst, its last one the end index into tcount (mark_needed
// turns the end into a count; tcount starts at 0, so empty leaves stay 0).
__global__ void k_target_ranges(const int* leaf, int64_t m, int* tfirst, int* tcount) {
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= m) return;
    const int b = leaf[i];
    if (i == 0 || leaf[i - 1] != b) tfirst[b] = (int)i;
    if (i == m - 1 || leaf[i + 1] != b) tcount[b] = (int)(i + 1);
}

void target_ranges(const int* leaf, int64_t m, int* tfirst, int* tcount, hipStream_t s) {
    if (m <= 0) return;
    k_target_ranges<<<nblocks(m, 256), 256, 0, s>>>(leaf, m, tfirst, tcount);
    SFMM_LAUNCH_CHECK();
}

// ------------------------------------------------------------------ walk
// Frontier form of Algorithm 1.  Each frontier pair (S, T) takes exactly
// one branch of INTERACTION(B_S, B_T); its recursive calls become the next
// frontier.  A source box without particles contributes nothing (it is a
// leaf, so no recursion is lost) and is dropped.
enum : uint8_t { A_NONE = 0, A_M2L = 1, A_P2P = 2, A_SPLIT_S = 3, A_SPLIT_T = 4, A_SPLIT_SELF = 5 };

// One round of the walk in three launches, sized on the device: the round's
// frontier size and output bases sit in st[0..2] (written by the previous
// round's emit), so rounds can be queued without reading anything back.  The
// pairs are taken in chunks of kWalkChunk, chunk c by workgroup c mod grid,
// in kWalkItems passes of kWalkThreads consecutive pairs (lane order = pair
// order).  k_walk_classify writes each pair's action and the chunk's three
// totals (children pairs, M2L pairs, P2P pairs); k_walk_chunk_scan scans the
// chunk totals; k_walk_emit scans the chunk's actions again and writes every
// output at its place in pair order, consecutive lanes to consecutive slots
// (so the lists come out in the same order as a scan over single pairs).
constexpr int kWalkItems = 4, kWalkThreads = 256, kWalkChunk = kWalkItems * kWalkThreads;

__device__ __forceinline__ int walk_nchild(uint8_t a) {
    return (a == A_SPLIT_S || a == A_SPLIT_T) ? 4 : (a == A_SPLIT_SELF ? 16 : 0);
}

// walk_action with the FP64 filters only: A_TIE where a double-double
// decision is needed (a MAC margin or a radius difference near zero)
constexpr uint8_t A_TIE = 7;
__device__ __forceinline__ uint8_t walk_action_fast(const WalkCtx& w, int s, int t) {
    const int2 bs = w.cc[s];
    if (bs.y == 0) return A_NONE;
    if (s == t) return (bs.x < 0) ? A_P2P : A_SPLIT_SELF;
    const int2 bt = w.cc[t];
    const double4 gs = w.geo[s], gt = w.geo[t];
    const double rs = gs.w, rt = gt.w;
    const int f = mac_far_filter_trig(gs.x, gs.y, gs.z, gt.x, gt.y, gt.z, protected_radius(rs, w.c_s, w.sigma), rt,
                                      w.strig[s], w.ttrig[t], 1.0, w.c_t);
    if (f > 0) return A_M2L;
    if (f == 0) return A_TIE;
    const bool sl = bs.x < 0, tl = bt.x < 0;
    if (!sl && !tl) {
        const double diff = rs - rt;
        if (!(fabs(diff) > 1e-13 * (rs + rt))) return A_TIE;
        return diff > 0.0 ? A_SPLIT_S : A_SPLIT_T;
    }
    if (!sl) return A_SPLIT_S;
    if (!tl) return A_SPLIT_T;
    return A_P2P;
}

// walk_action_fast's A_TIE cases decided exactly (double-double)
__device__ uint8_t walk_action_tie(const WalkCtx& w, int s, int t) {
    const int2 bs = w.cc[s], bt = w.cc[t];
    const double4 gs4 = w.geo[s], gt4 = w.geo[t];
    const double* a = w.gdd + 8 * (size_t)s;
    const double* b = w.gdd + 8 * (size_t)t;
    int f = mac_far_filter_trig(gs4.x, gs4.y, gs4.z, gt4.x, gt4.y, gt4.z, protected_radius(gs4.w, w.c_s, w.sigma),
                                gt4.w, w.strig[s], w.ttrig[t], 1.0, w.c_t);
    if (f == 0) {
        const dd csd[3] = {{a[0], a[1]}, {a[2], a[3]}, {a[4], a[5]}};
        const dd ctd[3] = {{b[0], b[1]}, {b[2], b[3]}, {b[4], b[5]}};
        const double* ta = w.dtrig + kWalkDtrig * (size_t)s;
        const double* tb = w.dtrig + kWalkDtrig * (size_t)t;
        const dd ts[2] = {{ta[0], ta[1]}, {ta[2], ta[3]}};
        const dd tt[4] = {{tb[4], tb[5]}, {tb[6], tb[7]}, {tb[8], tb[9]}, {tb[10], tb[11]}};
        f = mac_far_dd_trig(csd, ctd, dd{ta[12], ta[13]}, dd{b[6], b[7]}, ts, tt, 1.0, w.c_t) ? 1 : -1;
    }
    if (f > 0) return A_M2L;
    const bool sl = bs.x < 0, tl = bt.x < 0;
    if (!sl && !tl) return radius_greater(a[6], b[6], dd{a[6], a[7]}, dd{b[6], b[7]}) ? A_SPLIT_S : A_SPLIT_T;
    if (!sl) return A_SPLIT_S;
    if (!tl) return A_SPLIT_T;
    return A_P2P;
}

// Three counts of a thread summed over the workgroup (kWalkThreads):
// exclusive prefix in thread order (ex) and total (all).
__device__ __forceinline__ void walk_block_scan3(const int c[3], int (*sh)[kWalkThreads / 64], int ex[3], int all[3]) {
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    int x[3];
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        x[j] = c[j];
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int y = __shfl_up(x[j], o, 64);
            if (lane >= o) x[j] += y;
        }
        if (lane == 63) sh[j][wv] = x[j];
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        int before = 0, tot = 0;
#pragma unroll
        for (int v = 0; v < kWalkThreads / 64; ++v) {
            before += v < wv ? sh[j][v] : 0;
            tot += sh[j][v];
        }
        ex[j] = before + x[j] - c[j];
        all[j] = tot;
    }
    __syncthreads();  // sh is reused by the caller
}

// Classification of each chunk: FP64 decisions first; the near-ties of the
// chunk are gathered in LDS and decided exactly by consecutive threads (no
// wave runs that code for one lane); then the chunk's three totals.
__global__ void __launch_bounds__(kWalkThreads) k_walk_classify(const int2* __restrict__ F, const int* __restrict__ st,
                                                                WalkCtx w, uint8_t* __restrict__ action,
                                                                int* __restrict__ ctot, int cstride) {
    __shared__ int sh[3][kWalkThreads / 64];
    __shared__ int ntie;
    __shared__ short tie_at[kWalkChunk];
    __shared__ uint8_t tie_act[kWalkChunk];
    const int n = st[0];
    const int nchunk = (n + kWalkChunk - 1) / kWalkChunk;
    for (int ch = blockIdx.x; ch < nchunk; ch += gridDim.x) {
        const int k0 = ch * kWalkChunk;
        if (threadIdx.x == 0) ntie = 0;
        __syncthreads();
        uint8_t act[kWalkItems];
#pragma unroll
        for (int i = 0; i < kWalkItems; ++i) {
            const int li = i * kWalkThreads + threadIdx.x;
            act[i] = A_NONE;
            if (k0 + li < n) {
                const int2 f = F[k0 + li];
                act[i] = walk_action_fast(w, f.x, f.y);
                if (act[i] == A_TIE) tie_at[atomicAdd(&ntie, 1)] = (short)li;
            }
        }
        __syncthreads();
        for (int j = threadIdx.x; j < ntie; j += kWalkThreads) {
            const int li = tie_at[j];
            const int2 f = F[k0 + li];
            tie_act[li] = walk_action_tie(w, f.x, f.y);
        }
        __syncthreads();
        int c[3] = {0, 0, 0};
#pragma unroll
        for (int i = 0; i < kWalkItems; ++i) {
            const int li = i * kWalkThreads + threadIdx.x;
            if (k0 + li < n) {
                const uint8_t a = act[i] == A_TIE ? tie_act[li] : act[i];
                action[k0 + li] = a;
                c[0] += walk_nchild(a);
                c[1] += a == A_M2L;
                c[2] += a == A_P2P;
            }
        }
        int ex[3], all[3];
        walk_block_scan3(c, sh, ex, all);
        if (threadIdx.x == 0) {
#pragma unroll
            for (int j = 0; j < 3; ++j) ctot[(size_t)j * cstride + ch] = all[j];
        }
        // sh, ntie and the tie lists are reused by the next chunk (the scan
        // ends with a barrier)
    }
}

// exclusive scans of the three chunk-total arrays (one workgroup of
// kChunkScanThreads each, in pieces of that size with a running carry);
// tot[j] = the total of array j
constexpr int kChunkScanThreads = 1024;
__global__ void __launch_bounds__(kChunkScanThreads) k_walk_chunk_scan(const int* __restrict__ st,
                                                                       const int* __restrict__ ctot, int cstride,
                                                                       int* __restrict__ coff, int* __restrict__ tot) {
    constexpr int kWaves = kChunkScanThreads / 64;
    __shared__ int sh[kWaves];
    const int n = st[0];
    const int nchunk = (n + kWalkChunk - 1) / kWalkChunk;
    const int j = blockIdx.x;
    const int* in = ctot + (size_t)j * cstride;
    int* out = coff + (size_t)j * cstride;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    int carry = 0;
    for (int c0 = 0; c0 < nchunk; c0 += kChunkScanThreads) {
        const int i = c0 + threadIdx.x;
        const int v = i < nchunk ? in[i] : 0;
        int x = v;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int y = __shfl_up(x, o, 64);
            if (lane >= o) x += y;
        }
        if (lane == 63) sh[wv] = x;
        __syncthreads();
        int before = 0, all = 0;
#pragma unroll
        for (int q = 0; q < kWaves; ++q) {
            before += q < wv ? sh[q] : 0;
            all += sh[q];
        }
        if (i < nchunk) out[i] = carry + before + x - v;
        carry += all;
        __syncthreads();
    }
    if (threadIdx.x == 0) tot[j] = carry;
}

__device__ uint64_t pair_key(int s, int t) { return ((uint64_t)(uint32_t)t << 32) | (uint32_t)s; }

// Emit of one round.  The next frontier (tot[0] pairs) and the lists'
// new ends are checked against the capacities first: when anything would not
// fit, nothing is written, *overflow is set and the next round is empty (the
// caller then runs the walk again with room to spare).  Otherwise workgroup 0
// writes the next round's st (frontier size, M2L and P2P bases).
__global__ void __launch_bounds__(kWalkThreads) k_walk_emit(const int2* __restrict__ F, const int* __restrict__ st,
                                                            WalkCtx w, const uint8_t* __restrict__ action,
                                                            const int* __restrict__ coff, int cstride,
                                                            const int* __restrict__ tot, WalkCaps cap,
                                                            int2* __restrict__ Fnext, uint64_t* __restrict__ m2l,
                                                            uint64_t* __restrict__ p2p, int* __restrict__ st_next,
                                                            int* __restrict__ overflow) {
    __shared__ int sh[3][kWalkThreads / 64];
    const int n = st[0], bm = st[1], bp = st[2];
    const int nc = tot[0], am = tot[1], ap = tot[2];
    const bool fits = nc <= cap.frontier && (int64_t)bm + am <= cap.m2l && (int64_t)bp + ap <= cap.p2p;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        if (fits) {
            st_next[0] = nc;
            st_next[1] = bm + am;
            st_next[2] = bp + ap;
        } else {
            *overflow = 1;
            st_next[0] = 0;
            st_next[1] = bm;
            st_next[2] = bp;
        }
    }
    if (!fits) return;
    const int nchunk = (n + kWalkChunk - 1) / kWalkChunk;
    for (int ch = blockIdx.x; ch < nchunk; ch += gridDim.x) {
        const int k0 = ch * kWalkChunk;
        int oc = coff[ch];
        int om = bm + coff[(size_t)cstride + ch];
        int op = bp + coff[2 * (size_t)cstride + ch];
        for (int i = 0; i < kWalkItems && k0 + i * kWalkThreads < n; ++i) {  // uniform across the workgroup
            const int k = k0 + i * kWalkThreads + threadIdx.x;
            const uint8_t a = k < n ? action[k] : A_NONE;
            const int c[3] = {walk_nchild(a), a == A_M2L, a == A_P2P};
            int ex[3], all[3];
            walk_block_scan3(c, sh, ex, all);
            if (a != A_NONE) {
                const int s = F[k].x, t = F[k].y;
                int2* out = Fnext + oc + ex[0];
                switch (a) {
                    case A_M2L: m2l[om + ex[1]] = pair_key(s, t); break;
                    case A_P2P: p2p[op + ex[2]] = pair_key(s, t); break;
                    case A_SPLIT_S:
                        for (int q = 0; q < 4; ++q) out[q] = make_int2(w.cc[s].x + q, t);
                        break;
                    case A_SPLIT_T:
                        for (int q = 0; q < 4; ++q) out[q] = make_int2(s, w.cc[t].x + q);
                        break;
                    case A_SPLIT_SELF:
                        for (int q = 0; q < 4; ++q)
                            for (int r = 0; r < 4; ++r) out[4 * q + r] = make_int2(w.cc[s].x + q, w.cc[s].x + r);
                        break;
                    default: break;
                }
            }
            oc += all[0];
            om += all[1];
            op += all[2];
        }
    }
}

int walk_chunks(int n) {
    const int nchunk = (n + kWalkChunk - 1) / kWalkChunk;
    return nchunk > 0 ? nchunk : 1;
}

void walk_round_scan(const int2* F, const int* st, const WalkCtx& w, uint8_t* action, int* ctot, int* coff,
                     int cstride, int* tot, int grid, hipStream_t s) {
    k_walk_classify<<<grid, kWalkThreads, 0, s>>>(F, st, w, action, ctot, cstride);
    SFMM_LAUNCH_CHECK();
    k_walk_chunk_scan<<<3, kChunkScanThreads, 0, s>>>(st, ctot, cstride, coff, tot);
    SFMM_LAUNCH_CHECK();
}

void walk_round_emit(const int2* F, const int* st, const WalkCtx& w, const uint8_t* action, const int* coff,
                     int cstride, const int* tot, const WalkCaps& cap, int2* Fnext, uint64_t* m2l, uint64_t* p2p,
                     int* st_next, int* overflow, int grid, hipStream_t s) {
    k_walk_emit<<<grid, kWalkThreads, 0, s>>>(F, st, w, action, coff, cstride, tot, cap, Fnext, m2l, p2p, st_next,
                                             overflow);
    SFMM_LAUNCH_CHECK();
}

// ------------------------------------------------------------------ lists
// CSR offsets from the entries' target boxes in sorted order: off[b] = the
// first entry whose target is >= b
__global__ void k_csr_offsets(const int* tgt, int np, int nbox, int* off) {
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b > nbox) return;
    int lo = 0, hi = np;
    while (lo < hi) {
        const int mid = lo + ((hi - lo) >> 1);
        if (tgt[mid] < b) lo = mid + 1;
        else hi = mid;
    }
    off[b] = lo;
}

// source and target box of every entry from the sorted pair keys
__global__ void k_pair_split(const uint64_t* sorted, int np, int* src, int* tgt) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= np) return;
    const uint64_t v = sorted[k];
    src[k] = (int)(uint32_t)(v & 0xffffffffULL);
    tgt[k] = (int)(uint32_t)(v >> 32);
}

void pair_split(const uint64_t* sorted, int np, int* src, int* tgt, hipStream_t s) {
    if (np <= 0) return;
    k_pair_split<<<nblocks(np, 256), 256, 0, s>>>(sorted, np, src, tgt);
    SFMM_LAUNCH_CHECK();
}

void csr_offsets(const int* tgt, int np, int nbox, int* off, hipStream_t s) {
    k_csr_offsets<<<nblocks(nbox + 1, 256), 256, 0, s>>>(tgt, np, nbox, off);
    SFMM_LAUNCH_CHECK();
}

}  // namespace sfmm

// Sorts of (64-bit key, 32-bit value) pairs by the key, equal keys in the
// order given, without a pass over memory per digit (k_util.hip's radix sort:
// three launches per eight bits, 24 for a source's key): up to 8,192 pairs are
// sorted in one workgroup's LDS; more are first split by a sample's quantiles
// into buckets that fit there (five launches).
//
// Bound by the launches and by VALU issue: ranking takes ~55 instructions per
// 64 pairs and digit, of which a bucket needs five (block_sort).  Sorting the
// sources' keys, us of kernels, radix sort -> this: 1,000 pairs 110 -> 10,
// 10,000 112 -> 48, 1e6 170 -> 100, 1e7 870 -> 715; above 10,485,760 pairs the
// buckets, 2,048 at most, would outgrow one workgroup and the radix sort stays.
// Keys of up to 24 bits take it too (three passes at most, 17 us each at
// 786,432 targets against ~90 here).
#include "common.hpp"

namespace sfmm {

constexpr int kBsThreads = 1024, kBsWaves = kBsThreads / 64;
constexpr int kBsRounds = 16;                      // pairs per thread
constexpr int kBsCap = kBsThreads * kBsRounds;     // pairs of one workgroup: 128 KB of LDS
constexpr int kSampleMaxBuckets = 2048;

__device__ __forceinline__ uint64_t lanes_below(int lane) { return lane == 0 ? 0ULL : (~0ULL >> (64 - lane)); }

// Lanes of `among` that hold the same nbits-bit digit as this one
template <int NB>
__device__ __forceinline__ uint64_t same_digit(int d, uint64_t among, int nbits = NB) {
    uint32_t lo = (uint32_t)among, hi = (uint32_t)(among >> 32);
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        if (b >= nbits) break;
        const uint32_t mine = (uint32_t)__builtin_amdgcn_sbfe(d, b, 1);  // 0 or ~0
        const uint64_t m = __ballot(mine != 0);
        lo &= ~((uint32_t)m ^ mine);
        hi &= ~((uint32_t)(m >> 32) ^ mine);
    }
    return (uint64_t)hi << 32 | lo;
}

// Exclusive scan of one value per thread over the first 64 NW threads (every
// thread of the workgroup calls it; sh holds NW ints)
template <int NW>
__device__ __forceinline__ int scan_threads(int v, int* sh) {
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    int x = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int y = __shfl_up(x, o, 64);
        if (lane >= o) x += y;
    }
    if (lane == 63 && wv < NW) sh[wv] = x;
    __syncthreads();
    int before = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) before += w < wv ? sh[w] : 0;
    __syncthreads();  // sh may be reused
    return before + x - v;
}

constexpr int kBsIdBits = 14;  // a pair in LDS: window << 14 | index
constexpr int kBsWindow = 40;  // bits of the window (at most 50)
constexpr int kBsRunMax = 8;   // longest run of equal windows put in order pair by pair
static_assert(kBsCap == 1 << kBsIdBits && kBsWindow + kBsIdBits <= 64, "a pair is 64 bits");
constexpr uint64_t kBsId = kBsCap - 1;

template <int R>
struct BlockSort {
    uint64_t ex[kBsThreads * R];  // the pairs in order
    int cnt[kBsWaves][256];       // per-wave digit counts, then first slots
    int sh[8];
    uint32_t x[2];
};

// Stable sort of the workgroup's 1024 R pairs by the window's low `width`
// bits, eight at a time.  Thread t of wave v holds pairs v 64 R + 64 r + lane
// in e[r]; they end in the same places, and in ex.
template <int R>
__device__ __forceinline__ void sort_window(uint64_t* ex, int (*wcnt)[256], int* sh, uint64_t (&e)[R], int width) {
    const int t = threadIdx.x, wave = t >> 6, lane = t & 63;
    const int p0 = wave * 64 * R + lane;
    const uint64_t lt = lanes_below(lane);
    for (int shift = kBsIdBits; shift < kBsIdBits + width; shift += 8) {
#pragma unroll
        for (int k = 0; k < 256; k += 64) wcnt[wave][k + lane] = 0;  // read again by this wave alone
        int at[R];
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int d = (int)((e[r] >> shift) & 255);
            const uint64_t peers = same_digit<8>(d, ~0ULL);
            const int rank = __popcll(peers & lt);
            const int before = wcnt[wave][d];
            // every lane of the wave has read the count before its leader moves it
            __builtin_amdgcn_wave_barrier();
            if (rank == 0) wcnt[wave][d] = before + __popcll(peers);
            __builtin_amdgcn_wave_barrier();
            at[r] = before + rank;
            __builtin_amdgcn_sched_barrier(0);  // rounds interleaved hold more registers than there are
        }
        __syncthreads();
        int tot = 0;
        if (t < 256) {
#pragma unroll
            for (int v = 0; v < kBsWaves; ++v) tot += wcnt[v][t];
        }
        int run = scan_threads<4>(tot, sh);
        if (t < 256) {
#pragma unroll
            for (int v = 0; v < kBsWaves; ++v) {
                const int c = wcnt[v][t];
                wcnt[v][t] = run;
                run += c;
            }
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < R; ++r) ex[wcnt[wave][(e[r] >> shift) & 255] + at[r]] = e[r];
        __syncthreads();
#pragma unroll
        for (int r = 0; r < R; ++r) e[r] = ex[p0 + 64 * r];
    }
}

// Sorts cnt <= 1024 R keys, key(i) (masked to the bits to sort by): the low
// kBsIdBits bits of e[r] for place p = v 64 R + 64 r + lane become the index of
// the p-th key.  The places from cnt to 1024 R hold windows of ones, which stay
// behind the keys (the passes are stable).
//
// The keys are taken through the 40 bits below the highest one in which they
// differ: five passes.  Keys of one bucket seldom share these and differ below
// (a clustered sky of 1e6 points: 2 of 10,000, in runs of up to 3; with a window
// of 32 bits 3 of 100, runs up to 53).  Short runs are put in order pair by
// pair; where there is a long one, the bits below are sorted first and the
// window after them (at most 64 bits in all).
template <int R, class Key>
__device__ __forceinline__ void block_sort(uint64_t* ex, int (*wcnt)[256], int* sh, uint32_t* xr, uint64_t (&e)[R],
                                           int cnt, const Key& key) {
    const int t = threadIdx.x, wave = t >> 6, lane = t & 63;
    const int p0 = wave * 64 * R + lane;
    if (t < 2) xr[t] = 0;
    const uint64_t k0 = key(0);
    uint64_t x = 0;
#pragma unroll
    for (int r = 0; r < R; ++r) e[r] = p0 + 64 * r < cnt ? key(p0 + 64 * r) : k0;
#pragma unroll
    for (int r = 0; r < R; ++r) x |= e[r] ^ k0;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) x |= __shfl_xor(x, o, 64);
    __syncthreads();
    if (lane == 0) {
        atomicOr(&xr[0], (uint32_t)x);
        atomicOr(&xr[1], (uint32_t)(x >> 32));
    }
    __syncthreads();
    x = (uint64_t)xr[1] << 32 | xr[0];
    const int top = x == 0 ? 0 : 64 - __clzll((long long)x), low = max(0, top - kBsWindow);
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int p = p0 + 64 * r;
        e[r] = (p < cnt ? e[r] >> low << kBsIdBits : ~kBsId) | (uint64_t)p;
    }
    int width = min(top, kBsWindow);  // 0: all equal, in order
    for (int phase = 0;; ++phase) {  // the window; else the bits below it, then the window again
        sort_window<R>(ex, wcnt, sh, e, width);
        if (phase == 0) {
            if (low == 0) return;
            int longrun = 0, moved = 0;
            for (int p = t; p + 1 < cnt; p += kBsThreads) {
                const uint64_t w = ex[p];
                if ((w ^ ex[p + 1]) > kBsId || (p > 0 && (w ^ ex[p - 1]) <= kBsId)) continue;
                int hi = p + 1;  // p: the first of its run
                while (hi + 1 < cnt && hi - p < kBsRunMax && (w ^ ex[hi + 1]) <= kBsId) ++hi;
                if (hi - p >= kBsRunMax) {
                    longrun = 1;
                    continue;
                }
                for (int i = p + 1; i <= hi; ++i) {  // the windows of a run's places do not change
                    const uint64_t ei = ex[i], ki = key((int)(ei & kBsId));
                    int j = i;
                    for (; j > p && key((int)(ex[j - 1] & kBsId)) > ki; --j) ex[j] = ex[j - 1];
                    if (j < i) {
                        ex[j] = ei;
                        moved = 1;
                    }
                }
            }
            if (!__syncthreads_or(longrun)) {
                if (__syncthreads_or(moved)) {
#pragma unroll
                    for (int r = 0; r < R; ++r) e[r] = ex[p0 + 64 * r];
                }
                return;
            }
#pragma unroll
            for (int r = 0; r < R; ++r) {  // bits past the window's place fall off
                const int p = p0 + 64 * r;
                e[r] = (p < cnt ? key(p) << kBsIdBits : ~kBsId) | (uint64_t)p;
            }
            width = low;
        } else if (phase == 1) {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int id = (int)(e[r] & kBsId);
                e[r] = (id < cnt ? key(id) >> low << kBsIdBits : ~kBsId) | (uint64_t)id;
            }
            width = kBsWindow;
        } else {
            return;
        }
    }
}

// A bucket too large for LDS: one workgroup's passes over it in memory,
// between (ka, va) and (kb, vb); the result goes to (kb, vb).  off: 256 ints, the
// first free slot of each digit.
static __device__ void sort_large(int* off, int (*wcnt)[256], int* sh, uint64_t* ka, uint32_t* va, uint64_t* kb, uint32_t* vb, int64_t n,
                           uint64_t mask) {
    const int t = threadIdx.x, wave = t >> 6, lane = t & 63;
    uint64_t* const kout = kb;
    uint32_t* const vout = vb;
    for (int shift = 0; shift < 64; shift += 8) {
        if (((mask >> shift) & 255) == 0) break;
        if (t < 256) off[t] = 0;
        __syncthreads();
        for (int64_t i = t; i < n; i += kBsThreads) atomicAdd(&off[(ka[i] & mask) >> shift & 255], 1);
        __syncthreads();
        const int c = t < 256 ? off[t] : 0;
        const int first = scan_threads<4>(c, sh);
        if (t < 256) off[t] = first;
        for (int64_t i0 = 0; i0 < n; i0 += kBsThreads) {
#pragma unroll
            for (int k = 0; k < 256; k += 64) wcnt[wave][k + lane] = 0;
            __builtin_amdgcn_wave_barrier();
            const bool valid = i0 + t < n;
            const uint64_t key = valid ? ka[i0 + t] : 0;
            const uint32_t val = valid ? va[i0 + t] : 0u;
            const int d = (int)((key & mask) >> shift & 255);
            const uint64_t peers = same_digit<8>(d, __ballot(valid));
            const int rank = __popcll(peers & lanes_below(lane));
            if (valid && rank == 0) wcnt[wave][d] = __popcll(peers);
            __syncthreads();
            if (t < 256) {
                int run = off[t];
                for (int v = 0; v < kBsWaves; ++v) {
                    const int k = wcnt[v][t];
                    wcnt[v][t] = run;
                    run += k;
                }
                off[t] = run;
            }
            __syncthreads();
            if (valid) {
                const int pos = wcnt[wave][d] + rank;
                kb[pos] = key;
                vb[pos] = val;
            }
        }
        __syncthreads();  // with the writes above visible to the whole workgroup
        uint64_t* const k2 = ka;
        uint32_t* const v2 = va;
        ka = kb;
        va = vb;
        kb = k2;
        vb = v2;
    }
    if (ka != kout)
        for (int64_t i = t; i < n; i += kBsThreads) {
            kout[i] = ka[i];
            vout[i] = va[i];
        }
}

template <int R>
__device__ __forceinline__ void sort_pairs(uint64_t* ex, int (*wcnt)[256], int* sh, uint32_t* xr, const uint64_t* kin,
                                           const uint32_t* vin, uint64_t* kout, uint32_t* vout, int cnt,
                                           uint64_t mask) {
    uint64_t e[R], k[R];
    uint32_t v[R];
    block_sort<R>(ex, wcnt, sh, xr, e, cnt, [&](int i) { return kin[i] & mask; });
    const int p0 = (threadIdx.x >> 6) * 64 * R + (threadIdx.x & 63);
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int id = p0 + 64 * r < cnt ? (int)(e[r] & kBsId) : 0;
        k[r] = kin[id];
        v[r] = vin[id];
    }
    __syncthreads();  // in place: every pair is read before the first is written
#pragma unroll
    for (int r = 0; r < R; ++r) {
        if (p0 + 64 * r < cnt) {
            kout[p0 + 64 * r] = k[r];
            vout[p0 + 64 * r] = v[r];
        }
    }
}

// All n <= 1024 R pairs in one workgroup, in place
template <int R>
__global__ void __launch_bounds__(kBsThreads) k_sort_block(uint64_t* keys, uint32_t* vals, int n, uint64_t mask) {
    __shared__ BlockSort<R> S;
    sort_pairs<R>(S.ex, S.cnt, S.sh, S.x, keys, vals, keys, vals, n, mask);
}

// One workgroup per bucket.  spl: the splitters, whose equal neighbours mark a
// bucket of equal keys.
__global__ void __launch_bounds__(kBsThreads) k_sort_buckets(uint64_t* kin, uint32_t* vin, uint64_t* kout,
                                                             uint32_t* vout, uint64_t mask,
                                                             const int* __restrict__ bstart,
                                                             const uint64_t* __restrict__ spl) {
    __shared__ BlockSort<kBsRounds> S;
    const int b = blockIdx.x;
    const int base = bstart[b], cnt = bstart[b + 1] - base;
    if (cnt <= 0) return;
    kin += base;
    vin += base;
    kout += base;
    vout += base;
    if (b > 0 && b + 1 < (int)gridDim.x && spl[b - 1] == spl[b]) {  // equal keys only
        for (int i = threadIdx.x; i < cnt; i += kBsThreads) {
            kout[i] = kin[i];
            vout[i] = vin[i];
        }
        return;
    }
    const int R = (cnt + kBsThreads - 1) / kBsThreads;
    if (R > kBsRounds)
        sort_large(reinterpret_cast<int*>(S.ex), S.cnt, S.sh, kin, vin, kout, vout, cnt, mask);
    else if (R > 8)
        sort_pairs<kBsRounds>(S.ex, S.cnt, S.sh, S.x, kin, vin, kout, vout, cnt, mask);
    else if (R > 6)
        sort_pairs<8>(S.ex, S.cnt, S.sh, S.x, kin, vin, kout, vout, cnt, mask);
    else if (R > 4)
        sort_pairs<6>(S.ex, S.cnt, S.sh, S.x, kin, vin, kout, vout, cnt, mask);
    else if (R > 2)
        sort_pairs<4>(S.ex, S.cnt, S.sh, S.x, kin, vin, kout, vout, cnt, mask);
    else
        sort_pairs<2>(S.ex, S.cnt, S.sh, S.x, kin, vin, kout, vout, cnt, mask);
}

// Position i of ns = 2^lg_ns in a sample of n keys: the i-th of ns equal parts, at a
// pseudo-random place in it (splitmix64), so that no periodic order of the
// input misleads the quantiles
__device__ __forceinline__ int64_t sample_at(int i, int lg_ns, int64_t n) {
    uint64_t z = 0x9e3779b97f4a7c15ULL * (uint64_t)(i + 1);
    z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ULL;
    z = (z ^ (z >> 27)) * 0x94d049bb133111ebULL;
    z ^= z >> 31;
    const int64_t a = i * n >> lg_ns, e = (i + 1) * n >> lg_ns;  // ns <= n: not empty
    return a + (int64_t)((z >> 32) * (uint64_t)(e - a) >> 32);
}

// The nb - 1 quantiles of a sample of ns = 2^lg_ns <= 1024 R keys (a multiple of nb)
template <int R>
__global__ void __launch_bounds__(kBsThreads) k_sort_splitters(const uint64_t* __restrict__ kin, int64_t n, int lg_ns,
                                                               int nb, uint64_t mask, uint64_t* __restrict__ spl) {
    __shared__ BlockSort<R> S;
    uint64_t e[R];
    auto key = [&](int i) { return kin[sample_at(i, lg_ns, n)] & mask; };
    const int ns = 1 << lg_ns, step = ns / nb;
    block_sort<R>(S.ex, S.cnt, S.sh, S.x, e, ns, key);
    const int p0 = (threadIdx.x >> 6) * 64 * R + (threadIdx.x & 63);
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int p = p0 + 64 * r;
        if (p < ns && (p + 1) % step == 0 && (p + 1) / step < nb) spl[(p + 1) / step - 1] = key((int)(e[r] & kBsId));
    }
}

constexpr int kSplitRounds = 8;  // keys per thread of the splitting passes

// Bucket of every key of a tile (the first whose splitter is not below the
// key; the next one where that splitter occurs twice and the key equals it),
// and the tile's bucket counts, hist[bucket][tile]
template <int THREADS, int MAXB>
__global__ void __launch_bounds__(THREADS) k_sort_classify(const uint64_t* __restrict__ kin, int64_t n, int nb,
                                                           uint64_t mask, const uint64_t* __restrict__ spl, int rs,
                                                           uint16_t* __restrict__ bid, int* __restrict__ hist) {
    __shared__ uint64_t sp[MAXB];
    __shared__ int h[MAXB];
    const int64_t base = (int64_t)blockIdx.x * (THREADS * kSplitRounds);
    uint64_t k[kSplitRounds];
#pragma unroll
    for (int r = 0; r < kSplitRounds; ++r) {
        const int64_t i = base + r * THREADS + threadIdx.x;
        k[r] = i < n ? kin[i] & mask : 0;
    }
    for (int j = threadIdx.x; j < nb; j += THREADS) {
        sp[j] = j + 1 < nb ? spl[j] : 0;
        h[j] = 0;
    }
    __syncthreads();
    int b[kSplitRounds];
#pragma unroll
    for (int r = 0; r < kSplitRounds; ++r) b[r] = 0;
    for (int step = nb >> 1; step > 0; step >>= 1) {  // nb is a power of two
#pragma unroll
        for (int r = 0; r < kSplitRounds; ++r) b[r] += sp[b[r] + step - 1] < k[r] ? step : 0;
    }
#pragma unroll
    for (int r = 0; r < kSplitRounds; ++r) {
        const int64_t i = base + r * THREADS + threadIdx.x;
        if (i >= n) continue;
        if (b[r] + 2 < nb && sp[b[r]] == k[r] && sp[b[r] + 1] == k[r]) ++b[r];
        bid[i] = (uint16_t)b[r];
        atomicAdd(&h[b[r]], 1);
    }
    __syncthreads();
    for (int j = threadIdx.x; j < nb; j += THREADS) hist[(size_t)j * rs + blockIdx.x] = h[j];
}

// Stable scatter of a tile by its bucket numbers, through LDS so that each
// bucket's run is written as one piece (k_rs_scatter's way, with up to 2048
// buckets: the waves' counts are 16 bits wide and share the staged keys'
// memory).  The first tile writes the buckets' starts.
template <int THREADS, int MAXB>
__global__ void __launch_bounds__(THREADS) k_sort_split(const uint64_t* __restrict__ kin,
                                                        const uint32_t* __restrict__ vin, uint64_t* __restrict__ kout,
                                                        uint32_t* __restrict__ vout, int64_t n, int nb, int nbits,
                                                        int rs, const uint16_t* __restrict__ bid,
                                                        const int* __restrict__ offs, const int* __restrict__ dtot,
                                                        int* __restrict__ bstart) {
    constexpr int W = THREADS / 64, T = THREADS * kSplitRounds, PER = (MAXB + THREADS - 1) / THREADS;
    __shared__ union {
        uint16_t wcnt[W][MAXB];  // per-wave bucket counts, then each wave's first slot
        uint64_t sk[T];
    } u;
    __shared__ uint32_t sv[T];
    __shared__ uint16_t sb[T];
    __shared__ int goff[MAXB];  // global position of slot 0 of the tile's run of a bucket
    __shared__ int sh[W];
    const int t = threadIdx.x, wave = t >> 6, lane = t & 63;
    for (int j = lane; j < nb; j += 64) u.wcnt[wave][j] = 0;
    const int64_t tile0 = (int64_t)blockIdx.x * T, q0 = tile0 + wave * (64 * kSplitRounds);
    uint64_t key[kSplitRounds];
    uint32_t val[kSplitRounds];
    int d[kSplitRounds], at[kSplitRounds];
#pragma unroll
    for (int r = 0; r < kSplitRounds; ++r) {
        const int64_t i = q0 + r * 64 + lane;
        const bool valid = i < n;
        key[r] = valid ? kin[i] : 0;
        val[r] = valid ? vin[i] : 0u;
        d[r] = valid ? bid[i] : -1;
    }
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int r = 0; r < kSplitRounds; ++r) {
        const bool valid = d[r] >= 0;
        const int dd = valid ? d[r] : 0;
        const uint64_t peers = same_digit<11>(dd, __ballot(valid), nbits);
        const int rank = __popcll(peers & lanes_below(lane));
        const int before = u.wcnt[wave][dd];
        // every lane of the wave has read the count before its leader moves it
        __builtin_amdgcn_wave_barrier();
        if (valid && rank == 0) u.wcnt[wave][dd] = (uint16_t)(before + __popcll(peers));
        __builtin_amdgcn_wave_barrier();
        at[r] = before + rank;
    }
    __syncthreads();
    int tot[PER], gt[PER], sum = 0, gsum = 0;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int j = t * PER + k;
        tot[k] = gt[k] = 0;
        if (j < nb) {
            for (int w = 0; w < W; ++w) tot[k] += u.wcnt[w][j];
            gt[k] = dtot[j];
        }
        sum += tot[k];
        gsum += gt[k];
    }
    int lbase = scan_threads<W>(sum, sh), gbase = scan_threads<W>(gsum, sh);
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int j = t * PER + k;
        if (j < nb) {
            goff[j] = gbase + offs[(size_t)j * rs + blockIdx.x] - lbase;
            if (blockIdx.x == 0) {
                bstart[j] = gbase;
                if (j == nb - 1) bstart[nb] = (int)n;
            }
            int run = lbase;
            for (int w = 0; w < W; ++w) {
                const int c = u.wcnt[w][j];
                u.wcnt[w][j] = (uint16_t)run;
                run += c;
            }
        }
        lbase += tot[k];
        gbase += gt[k];
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kSplitRounds; ++r)
        if (d[r] >= 0) at[r] += u.wcnt[wave][d[r]];
    __syncthreads();  // the counts' memory now takes the keys
#pragma unroll
    for (int r = 0; r < kSplitRounds; ++r) {
        if (d[r] >= 0) {
            u.sk[at[r]] = key[r];
            sv[at[r]] = val[r];
            sb[at[r]] = (uint16_t)d[r];
        }
    }
    __syncthreads();
    const int cnt = (int)min((int64_t)T, n - tile0);
    for (int p = t; p < cnt; p += THREADS) {
        const int64_t pos = (int64_t)goff[sb[p]] + p;
        if (pos < 0 || pos >= n) continue;  // unreachable with consistent counts
        kout[pos] = u.sk[p];
        vout[pos] = sv[p];
    }
}

template <int THREADS, int MAXB>
static void sample_sort(uint64_t* keys, uint32_t* vals, uint64_t* kalt, uint32_t* valt, int64_t n, int nb, uint64_t mask,
                 hipStream_t s) {
    constexpr int T = THREADS * kSplitRounds;
    const int nt = (int)((n + T - 1) / T), rs = (nt + 3) & ~3;
    int nbits = 0;
    while ((1 << nbits) < nb) ++nbits;
    const int lg_ns = std::min(nbits + 4, kBsIdBits);
    uint64_t* spl = (uint64_t*)pool_alloc(sizeof(uint64_t) * nb);
    uint16_t* bid = (uint16_t*)pool_alloc(sizeof(uint16_t) * (size_t)n);
    int* hist = (int*)pool_alloc(sizeof(int) * (size_t)nb * rs);
    int* offs = (int*)pool_alloc(sizeof(int) * (size_t)nb * rs);
    int* dtot = (int*)pool_alloc(sizeof(int) * (2 * (size_t)nb + 1));
    int* bstart = dtot + nb;
    if (lg_ns <= 11)
        k_sort_splitters<2><<<1, kBsThreads, 0, s>>>(keys, n, lg_ns, nb, mask, spl);
    else if (lg_ns <= 12)
        k_sort_splitters<4><<<1, kBsThreads, 0, s>>>(keys, n, lg_ns, nb, mask, spl);
    else
        k_sort_splitters<kBsRounds><<<1, kBsThreads, 0, s>>>(keys, n, lg_ns, nb, mask, spl);
    SFMM_LAUNCH_CHECK();
    k_sort_classify<THREADS, MAXB><<<nt, THREADS, 0, s>>>(keys, n, nb, mask, spl, rs, bid, hist);
    SFMM_LAUNCH_CHECK();
    scan_rows(hist, nb, nt, rs, offs, dtot, s);
    k_sort_split<THREADS, MAXB><<<nt, THREADS, 0, s>>>(keys, vals, kalt, valt, n, nb, nbits, rs, bid, offs, dtot,
                                                       bstart);
    SFMM_LAUNCH_CHECK();
    k_sort_buckets<<<nb, kBsThreads, 0, s>>>(kalt, valt, keys, vals, mask, bstart, spl);
    SFMM_LAUNCH_CHECK();
    // freed blocks are only reused by later stream-ordered work on this stream
    pool_free(spl);
    pool_free(bid);
    pool_free(hist);
    pool_free(offs);
    pool_free(dtot);
}

bool sort_in_lds(int64_t n) { return n <= 8 * kBsThreads; }

bool sort_by_sample(int64_t n, int bits) { return n > 8 * kBsThreads && n <= kSampleSortMax && bits > kSampleMinBits; }

void block_sort_u64(uint64_t* keys, uint32_t* vals, int64_t n, int bits, hipStream_t s) {
    const uint64_t mask = bits >= 64 ? ~0ULL : (1ULL << bits) - 1;
    if (n <= 2 * kBsThreads)
        k_sort_block<2><<<1, kBsThreads, 0, s>>>(keys, vals, (int)n, mask);
    else if (n <= 4 * kBsThreads)
        k_sort_block<4><<<1, kBsThreads, 0, s>>>(keys, vals, (int)n, mask);
    else
        k_sort_block<8><<<1, kBsThreads, 0, s>>>(keys, vals, (int)n, mask);
    SFMM_LAUNCH_CHECK();
}

void sample_sort_u64(uint64_t* keys, uint32_t* vals, uint64_t* kalt, uint32_t* valt, int64_t n, int bits,
                     hipStream_t s) {
    const uint64_t mask = bits >= 64 ? ~0ULL : (1ULL << bits) - 1;
    int nb = 16;
    while (nb < kSampleMaxBuckets && (int64_t)nb * 4096 < n) nb *= 2;
    if (nb <= 512)
        sample_sort<256, 512>(keys, vals, kalt, valt, n, nb, mask, s);
    else
        sample_sort<1024, kSampleMaxBuckets>(keys, vals, kalt, valt, n, nb, mask, s);
}

}  // namespace sfmm

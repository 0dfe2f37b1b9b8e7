// Interaction lists of a plan (Algorithm 1, Sec. 3.4), pruned to the target
// side: only boxes that hold a target somewhere below them ever use a local
// expansion or a direct act, so only those get lists.  (The full lists of
// Algorithm 1, for every box, come from the frontier walk of k_tree.hip when
// the exports or the statistics ask for them.)
//
// The walk runs target by target instead of pair by pair.  A pair (S, T) that
// splits T hands S to T's four children, so the sources a box starts from are
// its parent's hand-down list D; a box whose pair with itself splits hands its
// own children down.  Level by level (k_group_walk<G_LEVEL>) the split boxes
// make D for the next level and count their FMM acts; then one launch counts
// the acts of all leaves that hold targets, and after a scan and one read-back
// of the totals one launch writes both lists straight into CSR order: no
// sorting by target, no frontier in memory.  A wave takes the four children
// of one split box together (they start from the same D): 64 (S, T) pairs a
// step, split sources go to a small stack in LDS.
//
// On clustered-1e7 with 3,145,728 grid targets (217,000 of 620,000 boxes hold
// one) the walk and the lists go from 3.1 ms of kernels (32 frontier rounds of
// three launches over every box, two sorts of 16 M pairs each, the near-field
// split) to 1.5 ms, and Lemma 3 over the pruned lists from 2.96 to 1.14 ms.
#include "common.hpp"
#include "geom.hpp"

#include <algorithm>

namespace sfmm {

static unsigned nblk(int64_t n, int b) { return (unsigned)((n + b - 1) / b > 0 ? (n + b - 1) / b : 1); }

// ------------------------------------------------------------ box records
// Geometry of every box and the walk's records of it in one pass: centre and
// scale, radius, the double-double forms for near-ties, and one 64-byte record
// (WalkRec) per source box, so that a lane's look at a source is one aligned
// segment.
// One lane a box is a serial chain of five pixel points, an angle and three
// sines in double-double, 27 us however few boxes there are.  kBoxLanes lanes
// share a box up to kBoxTeamMax boxes (three times the instructions, which
// the idle chip has room for): 27 -> 12 us up to 2,000 boxes, 28 -> 20 at
// 9,000, 27 -> 22 at 11,000, but 28 -> 32 at 17,000 and 45 -> 70 at 62,000.
constexpr int kBoxLanes = 8, kBoxTeamMax = 12288;

__device__ __forceinline__ dd shfl_dd(dd v, int lane, int width) {
    return {__shfl(v.hi, lane, width), __shfl(v.lo, lane, width)};
}

// box_geometry by the kBoxLanes lanes of one box (r: the lane's place among
// them): lanes 0 to 3 a vertex each, the others the centre, and the farthest
// vertex by comparisons in box_geometry's order, so the values are the same.
__device__ __forceinline__ BoxGeomDD box_geometry_team(int level, uint64_t pix, int r) {
    BoxGeomDD g;
    const double fx = r > 3 ? 0.5 : r == 1 || r == 2 ? 1.0 : 0.0, fy = r > 3 ? 0.5 : r >= 2 ? 1.0 : 0.0;
    dd v[3], far[3], ch = dd_from(0.0), best = dd_from(-1.0);
    pix_point_dd(level, pix, fx, fy, v);
    for (int i = 0; i < 3; ++i) {
        g.c[i] = shfl_dd(v[i], 4, kBoxLanes);
        const dd e = dd_sub(v[i], g.c[i]);
        ch = dd_add(ch, dd_mul(e, e));
    }
    int at = 0;
    for (int k = 0; k < 4; ++k) {
        const dd o = shfl_dd(ch, k, kBoxLanes);
        if (dd_lt(best, o)) {
            best = o;
            at = k;
        }
    }
    for (int i = 0; i < 3; ++i) far[i] = shfl_dd(v[i], at, kBoxLanes);
    g.r = angdist_dd(g.c, far);
    return g;
}

template <int LB>
__global__ void __launch_bounds__(128) k_box_records(int nb, const int* __restrict__ level,
                                                     const uint64_t* __restrict__ pixel,
                                                     const int* __restrict__ child0, const int* __restrict__ count,
                                                     double c_s, double c_t, double sigma, double ratio,
                                                     int min_count, double* __restrict__ cen,
                                                     double* __restrict__ rad, double* __restrict__ gdd,
                                                     WalkRec* __restrict__ rec, double4* __restrict__ ttrig,
                                                     double* __restrict__ dtrig, double* __restrict__ hfar) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const int b = i / LB, r8 = i % LB;
    if (b >= nb) return;  // uniform across a box's lanes
    const int L = level[b];
    BoxGeomDD g;
    if constexpr (LB == 1) g = box_geometry(L, pixel[b]);
    else g = box_geometry_team(L, pixel[b], r8);
    const double r = g.r.hi;
    const bool widen = sigma > 0.0 && r + sigma > c_s * r;
    const dd prot = widen ? dd_add(g.r, dd_from(sigma)) : dd_mul_d(g.r, c_s);
    const dd ang[3] = {prot, g.r, dd_div(g.r, dd_from(c_t))};
    double* t = dtrig + kWalkDtrig * (size_t)b;
    if constexpr (LB > 1) {
        // lanes 0 to 2 an angle each, the last lane what is left
        if (r8 < 3) {
            const dd x = r8 == 0 ? ang[0] : r8 == 1 ? ang[1] : ang[2];
            dd sn, cs;
            dd_sincos(x, &sn, &cs);
            t[4 * r8 + 0] = cs.hi;
            t[4 * r8 + 1] = cs.lo;
            t[4 * r8 + 2] = sn.hi;
            t[4 * r8 + 3] = sn.lo;
        }
        if (r8 != LB - 1) return;
    }
    cen[4 * (size_t)b + 0] = g.c[0].hi;
    cen[4 * (size_t)b + 1] = g.c[1].hi;
    cen[4 * (size_t)b + 2] = g.c[2].hi;
    cen[4 * (size_t)b + 3] = tan(0.5 * r);  // coefficient scale rho
    rad[b] = r;
    double* o = gdd + 8 * (size_t)b;
    o[0] = g.c[0].hi; o[1] = g.c[0].lo;
    o[2] = g.c[1].hi; o[3] = g.c[1].lo;
    o[4] = g.c[2].hi; o[5] = g.c[2].lo;
    o[6] = g.r.hi;    o[7] = g.r.lo;
    double s1, c1, s2, c2, s3, c3;
    sincos(protected_radius(r, c_s, sigma), &s1, &c1);
    sincos(r, &s2, &c2);
    sincos(r / c_t, &s3, &c3);
    WalkRec w;
    w.x = g.c[0].hi;
    w.y = g.c[1].hi;
    w.z = g.c[2].hi;
    w.r = r;
    w.cp = c1;
    w.sp = s1;
    w.child0 = child0[b];
    w.count = count[b];
    w.rlo = g.r.lo;
    rec[b] = w;
    ttrig[b] = make_double4(c2, s2, c3, s3);
    // chord beyond which the box is taken through its expansion at a target
    // (4: never): ratio R, and beyond every particle's profile
    const double a = fmax(ratio * r, r + sigma);
    hfar[b] = w.count >= min_count && a < 3.0 ? 2.0 * sin(0.5 * a) : 4.0;
    t[12] = prot.hi;
    t[13] = prot.lo;
    if constexpr (LB == 1) {
        for (int k = 0; k < 3; ++k) {
            dd sn, cs;
            dd_sincos(ang[k], &sn, &cs);
            t[4 * k + 0] = cs.hi;
            t[4 * k + 1] = cs.lo;
            t[4 * k + 2] = sn.hi;
            t[4 * k + 3] = sn.lo;
        }
    }
}

void box_records(int nb, const int* level, const uint64_t* pixel, const int* child0, const int* count,
                 double c_s, double c_t, double sigma, double ratio, int min_count, double* cen, double* rad,
                 double* gdd, WalkRec* rec, double4* ttrig, double* dtrig, double* hfar, hipStream_t s) {
    if (nb <= 0) return;
    if (nb <= kBoxTeamMax)
        k_box_records<kBoxLanes><<<nblk((int64_t)kBoxLanes * nb, 128), 128, 0, s>>>(
            nb, level, pixel, child0, count, c_s, c_t, sigma, ratio, min_count, cen, rad, gdd, rec, ttrig, dtrig, hfar);
    else
        k_box_records<1><<<nblk(nb, 128), 128, 0, s>>>(nb, level, pixel, child0, count, c_s, c_t, sigma, ratio,
                                                       min_count, cen, rad, gdd, rec, ttrig, dtrig, hfar);
    SFMM_LAUNCH_CHECK();
}

// ------------------------------------------------------------ boxes with targets
// tcount holds the end of each leaf's target run (k_target_ranges): turned
// into a count here, and the leaf and its ancestors are marked (a climb stops
// at a box that another one has marked: that one goes on to the root).
__global__ void k_mark_needed(const int* __restrict__ tfirst, int nbox, int* __restrict__ tcount,
                              const int* __restrict__ parent, uint8_t* need) {
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= nbox) return;
    const int e = tcount[b];
    if (e <= 0) return;
    tcount[b] = e - tfirst[b];
    volatile uint8_t* nd = need;
    for (int x = b; x >= 0 && !nd[x]; x = parent[x]) nd[x] = 1;
}

void mark_needed(const int* tfirst, int nbox, int* tcount, const int* parent, uint8_t* need, hipStream_t s) {
    if (nbox <= 0) return;
    k_mark_needed<<<nblk(nbox, 256), 256, 0, s>>>(tfirst, nbox, tcount, parent, need);
    SFMM_LAUNCH_CHECK();
}

// ------------------------------------------------------------ the walk
enum : uint8_t { A_NONE = 0, A_M2L = 1, A_P2P = 2, A_SPLIT_S = 3, A_SPLIT_T = 4, A_TIE = 7 };

// what a lane needs of its target box (in LDS, one of the group's four)
struct GroupTarget {
    double x, y, z, r, rlo;
    double4 trig;
    int child0;
};

// The branch of INTERACTION(B_S, B_T) for a pair that is neither empty nor a
// split box with itself.  The FP64 filter of the MAC decides nearly all;
// radii that agree to 1e-13 (congruent boxes, on the same ring for one: in
// most steps some lane meets them) are compared in double-double, in place;
// only an undecided MAC is left to group_action_tie.
__device__ __forceinline__ uint8_t split_side(bool sl, bool tl, double rs, double rslo, double rt, double rtlo) {
    if (!sl && !tl) return radius_greater(rs, rt, dd{rs, rslo}, dd{rt, rtlo}) ? A_SPLIT_S : A_SPLIT_T;
    if (!sl) return A_SPLIT_S;
    if (!tl) return A_SPLIT_T;
    return A_P2P;
}

__device__ __forceinline__ uint8_t group_action(const GroupCtx& w, const WalkRec& s, const GroupTarget& t) {
    const int f = mac_far_filter_trig(s.x, s.y, s.z, t.x, t.y, t.z, protected_radius(s.r, w.c_s, w.sigma), t.r,
                                      make_double2(s.cp, s.sp), t.trig, 1.0, w.c_t);
    if (f > 0) return A_M2L;
    if (f == 0) return A_TIE;
    return split_side(s.child0 < 0, t.child0 < 0, s.r, s.rlo, t.r, t.rlo);
}

// the double-double decision of a near-tie of the MAC (the context's pointers
// by value: a reference put the whole context into every lane's scratch memory
// at the kernel's start: a level kernel of 1e6 sources took 13 us instead of 9)
__device__ __noinline__ uint8_t group_action_tie(const WalkRec* rec, const double* gdd, const double* dtrig, double c_t,
                                                 int S, int T) {
    const WalkRec s = rec[S], t = rec[T];
    const double* a = gdd + 8 * (size_t)S;
    const double* b = gdd + 8 * (size_t)T;
    const dd csd[3] = {{a[0], a[1]}, {a[2], a[3]}, {a[4], a[5]}};
    const dd ctd[3] = {{b[0], b[1]}, {b[2], b[3]}, {b[4], b[5]}};
    const double* ta = dtrig + kWalkDtrig * (size_t)S;
    const double* tb = dtrig + kWalkDtrig * (size_t)T;
    const dd ts[2] = {{ta[0], ta[1]}, {ta[2], ta[3]}};
    const dd tt[4] = {{tb[4], tb[5]}, {tb[6], tb[7]}, {tb[8], tb[9]}, {tb[10], tb[11]}};
    if (mac_far_dd_trig(csd, ctd, dd{ta[12], ta[13]}, dd{b[6], b[7]}, ts, tt, 1.0, c_t)) return A_M2L;
    return split_side(s.child0 < 0, t.child0 < 0, s.r, s.rlo, t.r, t.rlo);
}

// A group is four sibling boxes 4G .. 4G + 3 (groups 0-2 are the base pixels,
// whose hand-down list is all twelve of them).  One workgroup of NW waves
// takes a group, or (SINGLE) one target of it.  Items are (S, q) pairs: first
// the hand-down list times the wanted targets, and the children of split
// sources on a stack in LDS (when it runs full the workgroup goes depth first,
// one item at a time, which grows it by at most 3 per level and so never
// beyond the kGroupSpare entries kept for it).
//   G_LEVEL: the group's split boxes with targets below: D of each, FMM acts counted
//   G_COUNT: its leaves with targets: FMM and direct acts counted (zeros for
//            boxes without targets)
//   G_FILL:  every box with targets: both lists
// Bound by the latency of a step (LDS pop, one 64-byte gather, ballots), not
// by its bytes: one wave per group and 32 groups a CU where there are many
// groups, four waves a group where a level has few (kGroupWide).  Two kinds of
// groups are queued (big) by the one-wave count and fill and taken by
// k_group_walk_big, eight waves to a target: those that would need more than
// kGroupSteps steps (a big leaf next to a dense clump meets every leaf of it:
// up to 7,300 direct acts on clustered-1e7, which kept single waves busy for
// 0.5 ms after all others had ended), and those with an undecided MAC, whose
// double-double code (TIE) would cost the one-wave kernels half their waves.
constexpr int kGroupSteps = 40, kGroupWide = 4096;
enum { G_LEVEL = 0, G_COUNT = 1, G_FILL = 2 };

template <int MODE, int NW, bool TIE, bool SINGLE>
__device__ __forceinline__ void group_walk(const GroupCtx& w, int G, int only, const GroupOut& o) {
    constexpr int kStep = 64 * NW, kStack = 1024 * NW, NT = SINGLE ? 1 : 4;
    __shared__ uint32_t stk[kStack];
    __shared__ GroupTarget tgt[4];
    __shared__ uint32_t s_want;
    // per wave: split sources, then FMM acts and D / direct acts per target
    __shared__ __align__(16) int wc[1 + 2 * NT][NW < 4 ? 4 : NW];
    const int tid = threadIdx.x, lane = tid & 63, wave = NW > 1 ? tid >> 6 : 0;
    const int T0 = 4 * G;
    bool want = false;
    int ch = -1;
    if (SINGLE) __syncthreads();  // the previous target's LDS reads have ended
    if (tid < 4) {
        const bool need = w.need[T0 + tid] != 0;
        const WalkRec r = w.rec[T0 + tid];
        ch = r.child0;
        want = need && (MODE == G_LEVEL ? ch >= 0 : MODE == G_COUNT ? ch < 0 : true);
        if (MODE == G_COUNT && !SINGLE) {
            const int T = T0 + tid;
            if (!need) o.mcnt[T] = 0;
            if (!want) o.pcnt[T] = 0;
            o.tflag[T] = want ? 1 : 0;
            o.nflag[T] = need ? 1 : 0;
        }
        if (SINGLE) want = want && tid == only;
        if (want) {
            GroupTarget& t = tgt[tid];
            t.x = r.x;
            t.y = r.y;
            t.z = r.z;
            t.r = r.r;
            t.rlo = r.rlo;
            t.trig = w.ttrig[T0 + tid];
            t.child0 = ch;
        }
        if (MODE == G_LEVEL && want) {
            // the box with itself splits: its own children come down first
            const int sp = (ch - 12) >> 2;
            int* out = o.dlist + (w.doff ? w.doff[sp] : (int64_t)sp * w.cd);
            for (int k = 0; k < 4; ++k)
                if (k < o.dcap) out[k] = ch + k;
        }
    }
    uint32_t wm;
    if (NW > 1) {
        const uint64_t b = __ballot(want);
        if (tid == 0) s_want = (uint32_t)b;
        __syncthreads();
        wm = s_want;
    } else {
        wm = (uint32_t)__ballot(want);
        __syncthreads();
    }
    if (wm == 0) return;
    const int nq = __popc(wm);
    uint32_t qs = 0;  // the wanted targets, two bits each
    for (int q = 3; q >= 0; --q)
        if (wm >> q & 1) qs = qs << 2 | (uint32_t)q;
    const int len = G < 3 ? 12 : w.doff ? w.dcnt[G - 3] : min(w.dcnt[G - 3], w.cd);
    const int* in = G < 3 ? nullptr : w.dlist + (w.doff ? w.doff[G - 3] : (int64_t)(G - 3) * w.cd);
    const int n_in = len * nq;
    // running counts per target: FMM acts; hand-down sources or direct acts
    int nm[NT], n2[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        nm[t] = 0;
        n2[t] = MODE == G_LEVEL ? 4 : 0;
    }
    int size = 0, pos = 0;
    const uint64_t lt = (1ull << lane) - 1;
    for (int step = 0; size > 0 || pos < n_in; ++step) {  // uniform across the workgroup
        const GroupTake take = group_take(size, n_in - pos, kStep, kStack);
        const int take_s = take.s, take_i = take.i;
        int S = 0, q = 0;
        const bool on = tid < take_s + take_i;
        if (tid < take_s) {
            const uint32_t code = stk[size - 1 - tid];
            S = (int)(code >> 2);
            q = (int)(code & 3);
        } else if (on) {
            const int it = pos + tid - take_s;
            const int e = it / nq, k = it - e * nq;
            q = (int)(qs >> (2 * k) & 3);
            S = in ? in[e] : e;
        }
        size -= take_s;
        pos += take_i;
        uint8_t act = A_NONE;
        int sch = -1;
        if (on) {
            const WalkRec r = w.rec[S];
            sch = r.child0;
            if (r.count == 0) {  // a source box without particles is dropped
            } else if (S == T0 + q) {
                act = sch < 0 ? A_P2P : A_NONE;
            } else {
                act = group_action(w, r, tgt[q]);
                if (TIE && act == A_TIE) act = group_action_tie(w.rec, w.gdd, w.dtrig, w.c_t, S, T0 + q);
            }
        }
        if (!TIE && (__ballot(act == A_TIE) || step == kGroupSteps)) {  // uniform (one wave)
            if (lane == 0) {
                o.big[1 + atomicAdd(o.big, 1)] = G;
                o.bigflag[G] = 1;
            }
            return;
        }
        constexpr uint8_t A2 = MODE == G_LEVEL ? A_SPLIT_T : A_P2P;
        const int slot = SINGLE ? 0 : q;
        const uint64_t ms = __ballot(act == A_SPLIT_S);
        uint64_t mm[NT], m2[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            mm[t] = __ballot(act == A_M2L && slot == t);
            m2[t] = __ballot(act == A2 && slot == t);
        }
        int bs = size, bm[NT], b2[NT];  // where this wave's outputs start
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            bm[t] = nm[t];
            b2[t] = n2[t];
        }
        if constexpr (NW > 1) {
            if (lane == 0) {
                wc[0][wave] = __popcll(ms);
#pragma unroll
                for (int t = 0; t < NT; ++t) {
                    wc[1 + t][wave] = __popcll(mm[t]);
                    wc[1 + NT + t][wave] = __popcll(m2[t]);
                }
            }
            __syncthreads();  // every pop read, every count written
            int before[1 + 2 * NT], all[1 + 2 * NT];
#pragma unroll
            for (int k = 0; k < 1 + 2 * NT; ++k) {
                before[k] = all[k] = 0;
#pragma unroll
                for (int v = 0; v < NW; v += 4) {
                    const int4 x = *reinterpret_cast<const int4*>(&wc[k][v]);
                    before[k] += (v + 0 < wave ? x.x : 0) + (v + 1 < wave ? x.y : 0) + (v + 2 < wave ? x.z : 0) +
                                 (v + 3 < wave ? x.w : 0);
                    all[k] += x.x + x.y + x.z + x.w;
                }
            }
            bs += 4 * before[0];
            size += 4 * all[0];
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                bm[t] += before[1 + t];
                b2[t] += before[1 + NT + t];
                nm[t] += all[1 + t];
                n2[t] += all[1 + NT + t];
            }
        } else {
            __syncthreads();  // every pop read
            size += 4 * __popcll(ms);
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                nm[t] += __popcll(mm[t]);
                n2[t] += __popcll(m2[t]);
            }
        }
        if (act == A_SPLIT_S) {
            const int at = bs + 4 * __popcll(ms & lt);
#pragma unroll
            for (int k = 0; k < 4; ++k) stk[at + k] = (uint32_t)(sch + k) << 2 | (uint32_t)q;
        }
        if (MODE == G_FILL && act == A_M2L) {
            uint64_t m = mm[0];
            int b = bm[0];
#pragma unroll
            for (int t = 1; t < NT; ++t) {
                m = slot == t ? mm[t] : m;
                b = slot == t ? bm[t] : b;
            }
            const int at = o.moff[T0 + q] + b + __popcll(m & lt);
            o.msrc[at] = S;
            if (o.ment) o.ment[at] = T0 + q;
        }
        if (MODE != G_COUNT && act == A2) {
            uint64_t m = m2[0];
            int b = b2[0];
#pragma unroll
            for (int t = 1; t < NT; ++t) {
                m = slot == t ? m2[t] : m;
                b = slot == t ? b2[t] : b;
            }
            const int at = b + __popcll(m & lt);
            if (MODE == G_FILL) {
                o.psrc[o.poff[T0 + q] + at] = S;
            } else if (at < o.dcap) {
                const int sp = (tgt[q].child0 - 12) >> 2;
                o.dlist[(w.doff ? w.doff[sp] : (int64_t)sp * w.cd) + at] = S;
            }
        }
        __syncthreads();  // the pushes are visible to the next pops
    }
    if (MODE == G_FILL) return;
    if (tid < 4 && want) {
        const int T = T0 + tid;
        int km = nm[0], k2 = n2[0];
#pragma unroll
        for (int t = 1; t < NT; ++t) {
            km = tid == t ? nm[t] : km;
            k2 = tid == t ? n2[t] : k2;
        }
        o.mcnt[T] = km;
        if (MODE == G_COUNT) {
            o.pcnt[T] = k2;
        } else {
            o.dcnt[(ch - 12) >> 2] = k2;
            if (k2 > o.dcap) atomicMax(o.dmax, k2);
        }
    }
}

template <int NW>
__global__ void __launch_bounds__(64 * NW) k_group_level(GroupCtx w, int G0, GroupOut o) {
    group_walk<G_LEVEL, NW, true, false>(w, G0 + blockIdx.x, 0, o);
}

template <int MODE>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(8))) k_group_walk(GroupCtx w, GroupOut o) {
    const int G = blockIdx.x;
    if (MODE == G_FILL && o.bigflag[G]) return;
    if (MODE == G_COUNT && threadIdx.x == 0) o.bigflag[G] = 0;
    group_walk<MODE, 1, false, false>(w, G, 0, o);
}

// the queued groups (any order: each target is written by one workgroup)
template <int MODE>
__global__ void __launch_bounds__(512) k_group_walk_big(GroupCtx w, GroupOut o) {
    const int n = 4 * o.big[0];
    for (int j = blockIdx.x; j < n; j += gridDim.x) group_walk<MODE, 8, true, true>(w, o.big[1 + (j >> 2)], j & 3, o);
}

void group_walk_level(const GroupCtx& w, const GroupOut& o, int box0, int box1, hipStream_t s) {
    if (box1 <= box0) return;
    const int ng = (box1 - box0) / 4;
    if (ng <= kGroupWide) k_group_level<4><<<ng, 256, 0, s>>>(w, box0 / 4, o);
    else k_group_level<1><<<ng, 64, 0, s>>>(w, box0 / 4, o);
    SFMM_LAUNCH_CHECK();
}

static int big_grid(int ng) { return std::min(4 * ng, 1024); }

void group_walk_count(const GroupCtx& w, const GroupOut& o, int nbox, hipStream_t s) {
    if (nbox <= 0) return;
    const int ng = nbox / 4;
    k_group_walk<G_COUNT><<<ng, 64, 0, s>>>(w, o);
    SFMM_LAUNCH_CHECK();
    k_group_walk_big<G_COUNT><<<big_grid(ng), 512, 0, s>>>(w, o);
    SFMM_LAUNCH_CHECK();
}

void group_walk_fill(const GroupCtx& w, const GroupOut& o, int nbox, hipStream_t s) {
    if (nbox <= 0) return;
    const int ng = nbox / 4;
    k_group_walk<G_FILL><<<ng, 64, 0, s>>>(w, o);
    SFMM_LAUNCH_CHECK();
    k_group_walk_big<G_FILL><<<big_grid(ng), 512, 0, s>>>(w, o);
    SFMM_LAUNCH_CHECK();
}

// After the scan of the four per-box counts (FMM acts, direct acts, leaf with
// targets, box with targets): the leaves with targets as a list, and the
// sizes the host needs, written to its pinned memory (no copy launches):
// out[0..3] the totals, [4] the longest hand-down list if one did not fit,
// [5] the boxes with targets before box lc1 (the precision tier's FP64 ones).
__global__ void k_target_leaves(const int* __restrict__ tflag, const int* __restrict__ toff,
                                const int* __restrict__ noff, int nbox, int lc1, const int* __restrict__ tot,
                                const int* __restrict__ dmax, const int* __restrict__ pcnt, int* __restrict__ tl,
                                int* __restrict__ moff, int* __restrict__ poff, int* __restrict__ out) {
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b < nbox && tflag[b]) {
        tl[toff[b]] = b;
        if (pcnt[b] > kOneGroupList) __hip_atomic_store(out + 6, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
    if (b == 0) {
        for (int k = 0; k < 4; ++k) out[k] = tot[k];
        out[4] = *dmax;
        out[5] = lc1 < nbox ? noff[lc1] : tot[3];
        moff[nbox] = tot[0];  // the CSR ends
        poff[nbox] = tot[1];
    }
}

void target_leaves(const int* tflag, const int* toff, const int* noff, int nbox, int lc1, const int* tot,
                   const int* dmax, const int* pcnt, int* tl, int* moff, int* poff, int* out, hipStream_t s) {
    k_target_leaves<<<nblk(nbox, 256), 256, 0, s>>>(tflag, toff, noff, nbox, lc1, tot, dmax, pcnt, tl, moff, poff,
                                                    out);
    SFMM_LAUNCH_CHECK();
}

// M2L order keys of the boxes with targets: boxes of levels <= lc first (bit
// 7 clear), most team rounds first within each part (an 8-bit key: lists of
// 127 rounds or more share the first bucket), box order within a bucket.
__global__ void k_m2l_keys(const int* __restrict__ moff, const int* __restrict__ nflag, const int* __restrict__ noff,
                           const int* __restrict__ level, int lc, int tw_coarse, int tw_fine, int nbox,
                           uint64_t* __restrict__ keys, uint32_t* __restrict__ vals) {
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= nbox || !nflag[b]) return;
    const bool fine = level[b] > lc;
    const int tw = fine ? tw_fine : tw_coarse;
    const int rounds = (moff[b + 1] - moff[b] + tw - 1) / tw;
    const int at = noff[b];
    keys[at] = (uint64_t)((fine ? 128 : 0) | (127 - min(rounds, 127)));
    vals[at] = (uint32_t)b;
}

void m2l_keys(const int* moff, const int* nflag, const int* noff, const int* level, int lc, int tw_coarse,
              int tw_fine, int nbox, uint64_t* keys, uint32_t* vals, hipStream_t s) {
    if (nbox <= 0) return;
    k_m2l_keys<<<nblk(nbox, 256), 256, 0, s>>>(moff, nflag, noff, level, lc, tw_coarse, tw_fine, nbox, keys, vals);
    SFMM_LAUNCH_CHECK();
}

// ------------------------------------------------------------ direct-act lists
// Each leaf's direct acts are split in two: entries taken particle by
// particle from the front of its CSR run, entries taken through their Lemma 1
// expansion from its end, nn[T] of the first kind.
//
// With ORDERED (the precision tier) they are first put in Algorithm 1's own
// order (the round in which the frontier walk emits the pair, then the
// source's place along the sphere's key order): the tier's FP32 sums over
// tiles of 128 particles depend on it.  The FP64 sums do not (beyond their
// rounding), and keep the walk's own order, which is as reproducible.
//
// The round of (S, T) is level(S) + level(T) less the self splits above it
// (one per common ancestor: a self split lowers both levels in one round), so
// within one T it orders like level(S) - (common ancestors).  Two sources of
// the same round diverge at a common parent whose children are taken in pixel
// order: the first particle index orders them (sources of one list are
// disjoint and not empty).
__device__ __forceinline__ int common_levels(uint64_t ka, uint64_t kb) {
    // number of levels at which two order-29 keys share a pixel (0: other base pixels)
    const uint64_t x = ka ^ kb;
    return x == 0 ? 30 : max(0, 29 - (63 - (int)__clzll((long long)x)) / 2);
}

__device__ __forceinline__ uint64_t box_key(const NearCtx& c, int b) {
    return c.pixel[b] << (2 * (kOrder - c.level[b]));
}

__device__ __forceinline__ uint64_t act_key(const NearCtx& c, int S, int T, uint64_t kt) {
    const int ls = c.level[S];
    const int self = S == T ? ls : common_levels(c.pixel[S] << (2 * (kOrder - ls)), kt);
    return act_order_key(ls - self + 32, c.first[S]);  // a round of 2 .. 61
}

// the 64-bit value of lane j (uniform) in scalar registers
__device__ __forceinline__ uint64_t lane_u64(uint64_t v, int j) {
    const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)v, j), hi = __builtin_amdgcn_readlane((uint32_t)(v >> 32), j);
    return (uint64_t)hi << 32 | lo;
}

__device__ __forceinline__ double lane_f64(double v, int j) {
    return __longlong_as_double((long long)lane_u64((uint64_t)__double_as_longlong(v), j));
}

// S (live lanes) goes through its expansion at every target of T: all of them
// farther (as chords) than hfar[S] from its centre.  Every target lies within
// R_T of T's centre, so a centre distance beyond hfar + R_T settles it, and
// one below hfar - R_T settles the opposite.  Of the entries in between and the
// targets, the fewer are taken one after another and the others by the lanes:
// few targets each against all entries, or an entry against 64 targets a step
// until one is too close.  (Targets one after another at any number of them:
// 2,001 sources at 1.5e6 targets 2,364 us instead of 180; entries at any
// number: the longest lists of clustered-1e7 106 -> 125 us.)
__device__ __forceinline__ bool act_far(const NearCtx& c, bool live, int S, const WalkRec& t, int t0, int nt) {
    const double h = live ? c.hfar[S] : 4.0;
    bool far = false, open = false;
    WalkRec s{};
    if (h <= 2.0) {
        s = c.rec[S];
        const double ex = s.x - t.x, ey = s.y - t.y, ez = s.z - t.z;
        const double d2 = ex * ex + ey * ey + ez * ez;
        const double hi = h + t.r, lo = h - t.r;
        far = d2 > hi * hi * (1.0 + 1e-12);
        open = !far && !(lo > 0.0 && d2 < lo * lo * (1.0 - 1e-12));
    }
    const double thr = h * h;
    uint64_t left = __ballot(open);
    if (left == 0) return far;
    const int lane = threadIdx.x & 63;
    double nx = 0.0, ny = 0.0, nz = 0.0;
    auto load = [&](int b) {
        const int i = t0 + min(b + lane, nt - 1);
        nx = c.tx[i];
        ny = c.ty[i];
        nz = c.tz[i];
    };
    if (nt > 0) load(0);
    if (nt < __popcll(left)) {  // below 64
        for (int k = 0; k < nt; ++k) {
            const double dx = lane_f64(nx, k) - s.x, dy = lane_f64(ny, k) - s.y, dz = lane_f64(nz, k) - s.z;
            open = open && dx * dx + dy * dy + dz * dz > thr;
        }
        return far || open;
    }
    for (int b = 0; b < nt && left; b += 64) {  // uniform across the wave
        const double x = nx, y = ny, z = nz;
        if (b + 64 < nt) load(b + 64);
        for (uint64_t w = left; w; w &= w - 1) {
            const int j = __builtin_ctzll(w);
            const double dx = x - lane_f64(s.x, j), dy = y - lane_f64(s.y, j), dz = z - lane_f64(s.z, j);
            if (__ballot(!(dx * dx + dy * dy + dz * dz > lane_f64(thr, j)))) left &= ~(1ull << j);
        }
    }
    return far || (left >> lane & 1);
}

// Lists of up to kShortRanked (ordered) or kShortPlain entries: a wave each.
// An ordered list's keys sit in registers, four to a lane, and every entry's
// rank is counted against each key in turn.  Longer lists are queued for
// k_near_long, in two queues of 1 + ntl ints: up to kMidList entries, and more.
// Lists of more than kOneGroupList entries go to a third one (huge): their
// entries, their number, then the leaf and the first of its places among the
// entries of all of them.
constexpr int kShortRanked = 256, kShortPlain = 512, kMidList = 1024;
template <bool ORDERED>
__global__ void __launch_bounds__(256) k_near_short(NearCtx c, const int* __restrict__ tl, int ntl,
                                                    const int* __restrict__ poff, const int* __restrict__ praw,
                                                    int* __restrict__ psrc, int* __restrict__ nn,
                                                    int* __restrict__ queue, int* __restrict__ huge) {
    const int i = (int)((blockIdx.x * (int64_t)blockDim.x + threadIdx.x) >> 6);
    const int lane = threadIdx.x & 63;
    if (i >= ntl) return;  // uniform across the wave
    const int T = tl[i], k0 = poff[T], n = poff[T + 1] - k0;
    if (n > (ORDERED ? kShortRanked : kShortPlain)) {
        if (lane == 0) {
            if (n > kOneGroupList) {
                // number and first place together: list j's entries lie behind
                // those of the lists before it, as the sort by j leaves them
                const unsigned long long at =
                    atomicAdd(reinterpret_cast<unsigned long long*>(huge), (1ull << 32) | (unsigned)n);
                const int j = (int)(at >> 32);
                huge[2 + 2 * j] = T;
                huge[3 + 2 * j] = (int)(uint32_t)at;
            } else {
                int* q = n <= kMidList ? queue : queue + 1 + ntl;
                q[1 + atomicAdd(q, 1)] = T;
            }
        }
        return;
    }
    const WalkRec t = c.rec[T];
    const int t0 = c.tfirst[T], nt = c.tcount[T];
    const uint64_t lt = (1ull << lane) - 1;
    int bn = 0, bf = 0;  // near and far entries placed
    if constexpr (ORDERED) {
        constexpr int K = kShortRanked / 64;
        const uint64_t kt = box_key(c, T);
        uint64_t key[K];
        int S[K], rank[K], rfar[K];
        uint64_t fm[K];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int e = 64 * k + lane;
            key[k] = ~0ull;
            rank[k] = rfar[k] = S[k] = 0;
            if (e < n) {
                S[k] = praw[k0 + e];
                key[k] = act_key(c, S[k], T, kt);
            }
            fm[k] = 64 * k < n ? __ballot(act_far(c, e < n, S[k], t, t0, nt)) : 0;
            bf += __popcll(fm[k]);
        }
#pragma unroll
        for (int k = 0; k < K; ++k) {
            for (int j = 0; j < min(64, n - 64 * k); ++j) {
                const uint64_t kj = lane_u64(key[k], j);
                const int fj = (int)(fm[k] >> j & 1);
#pragma unroll
                for (int m = 0; m < K; ++m) {
                    if (64 * m >= n) break;  // uniform
                    const bool lower = kj < key[m];
                    rank[m] += lower;
                    rfar[m] += lower ? fj : 0;
                }
            }
        }
#pragma unroll
        for (int k = 0; k < K; ++k) {
            if (64 * k + lane >= n) continue;
            const bool far = fm[k] >> lane & 1;
            psrc[k0 + (far ? n - 1 - rfar[k] : rank[k] - rfar[k])] = S[k];
        }
        bn = n - bf;
    } else {
        for (int e0 = 0; e0 < n; e0 += 64) {
            const bool live = e0 + lane < n;
            const int S = live ? praw[k0 + e0 + lane] : 0;
            const bool far = act_far(c, live, S, t, t0, nt), near = live && !far;
            const uint64_t mn = __ballot(near), mf = __ballot(far);
            if (near) psrc[k0 + bn + __popcll(mn & lt)] = S;
            if (far) psrc[k0 + n - 1 - bf - __popcll(mf & lt)] = S;
            bn += __popcll(mn);
            bf += __popcll(mf);
        }
    }
    if (lane == 0) nn[T] = bn;
}

// Longer lists: a workgroup each (256 threads up to kMidList entries, 1024
// beyond).  Ordered, up to CAP entries: the keys (with the entry's place in the
// raw list) go through a bitonic network in LDS.  The network keeps the smaller
// key at the lower place in every comparator (mirrored first step), so places
// past the end never take part.
template <bool ORDERED, int kLongThreads, int CAP>
__global__ void __launch_bounds__(kLongThreads) k_near_long(NearCtx c, const int* __restrict__ poff,
                                                            const int* __restrict__ praw, int* __restrict__ psrc,
                                                            int* __restrict__ nn, const int* __restrict__ queue) {
    __shared__ uint64_t key[ORDERED ? CAP : 1];
    __shared__ int wsum[2][kLongThreads / 64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint64_t lt = (1ull << lane) - 1;
    const int nl = queue[0];
    for (int j = blockIdx.x; j < nl; j += gridDim.x) {
        const int T = queue[1 + j], k0 = poff[T], n = poff[T + 1] - k0;
        const int* raw = praw + k0;
        const WalkRec t = c.rec[T];
        if constexpr (ORDERED) {
            const uint64_t kt = box_key(c, T);
            for (int e = tid; e < n; e += kLongThreads) key[e] = act_key(c, raw[e], T, kt) << kActPlaceBits | (uint64_t)e;
            __syncthreads();
            for (int lk = 1; (1 << (lk - 1)) < n; ++lk) {
                for (int lh = lk; lh > 0; --lh) {
                    // blocks of 2^lh: at lh == lk the partner is mirrored in its
                    // block, then half-cleaners
                    const int hm = (1 << (lh - 1)) - 1;  // half block less one
                    for (int p = tid; p < (n + 1) / 2 + hm + 1; p += kLongThreads) {
                        const int r = p & hm, a = ((p & ~hm) << 1) + r;
                        const int b = lh == lk ? a + 2 * (hm - r) + 1 : a + hm + 1;
                        if (b < n) {
                            const uint64_t ka = key[a], kb = key[b];
                            if (kb < ka) {
                                key[a] = kb;
                                key[b] = ka;
                            }
                        }
                    }
                    __syncthreads();
                }
            }
        }
        int bn = 0, bf = 0;
        const int t0 = c.tfirst[T], nt = c.tcount[T];
        for (int base = 0; base < n; base += kLongThreads) {
            const int e = base + tid;
            const bool live = e < n;
            const int S = live ? raw[ORDERED ? (int)(key[e] & ((1u << kActPlaceBits) - 1)) : e] : 0;
            const bool far = act_far(c, live, S, t, t0, nt), near = live && !far;
            const uint64_t mn = __ballot(near), mf = __ballot(far);
            if (lane == 0) {
                wsum[0][wave] = __popcll(mn);
                wsum[1][wave] = __popcll(mf);
            }
            __syncthreads();
            int pn = bn + __popcll(mn & lt), pf = bf + __popcll(mf & lt);
            for (int v = 0; v < kLongThreads / 64; ++v) {
                pn += v < wave ? wsum[0][v] : 0;
                pf += v < wave ? wsum[1][v] : 0;
                bn += wsum[0][v];
                bf += wsum[1][v];
            }
            if (near) psrc[k0 + pn] = S;
            if (far) psrc[k0 + n - 1 - pf] = S;
            __syncthreads();  // wsum (and the keys) are reused
        }
        if (tid == 0) nn[T] = bn;
    }
}

// The huge lists are taken by the whole chip, entry by entry: sort keys (ordered;
// list j's number above the order's key) and one sort of them all, then the far
// flags, a scan of these over all lists, and every entry to its place.  By one
// workgroup each, lists of 1e5 to 2.6e5 entries took 4 ms and more for their
// network and 16 ms for the flags against 600 targets (1e6 sources of one clump
// in leaves of 8); here some 0.4 ms each.
// blockIdx.x: the list; vals null: the entries as they were made
struct HugeList {
    int T, base, k0, n;
};
__device__ __forceinline__ HugeList huge_list(const int* __restrict__ huge, const int* __restrict__ poff) {
    const int T = huge[2 + 2 * blockIdx.x], k0 = poff[T];
    return {T, huge[3 + 2 * blockIdx.x], k0, poff[T + 1] - k0};
}

__global__ void __launch_bounds__(256) k_huge_keys(NearCtx c, const int* __restrict__ poff,
                                                   const int* __restrict__ praw, const int* __restrict__ huge,
                                                   uint64_t* __restrict__ keys, uint32_t* __restrict__ vals) {
    const HugeList l = huge_list(huge, poff);
    const uint64_t kt = box_key(c, l.T);
    for (int e = blockIdx.y * 256 + threadIdx.x; e < l.n; e += 256 * gridDim.y) {
        const int S = praw[l.k0 + e];
        keys[l.base + e] = (uint64_t)blockIdx.x << kActKeyBits | act_key(c, S, l.T, kt);
        vals[l.base + e] = (uint32_t)S;
    }
}

__global__ void __launch_bounds__(256) k_huge_flags(NearCtx c, const int* __restrict__ poff,
                                                    const int* __restrict__ praw, const int* __restrict__ huge,
                                                    const uint32_t* __restrict__ vals, int* __restrict__ far) {
    const HugeList l = huge_list(huge, poff);
    const WalkRec t = c.rec[l.T];
    const int t0 = c.tfirst[l.T], nt = c.tcount[l.T];
    for (int e0 = blockIdx.y * 256; e0 < l.n; e0 += 256 * gridDim.y) {  // uniform across the workgroup
        const int e = e0 + threadIdx.x;
        const bool live = e < l.n;
        const int S = !live ? 0 : vals ? (int)vals[l.base + e] : praw[l.k0 + e];
        const bool f = act_far(c, live, S, t, t0, nt);
        if (live) far[l.base + e] = f ? 1 : 0;
    }
}

// before [ne + 1]: far entries before each one of all the lists', then their number
__global__ void __launch_bounds__(256) k_huge_place(const int* __restrict__ poff, const int* __restrict__ praw,
                                                    const int* __restrict__ huge, const uint32_t* __restrict__ vals,
                                                    const int* __restrict__ far, const int* __restrict__ before,
                                                    int* __restrict__ psrc, int* __restrict__ nn) {
    const HugeList l = huge_list(huge, poff);
    const int b0 = before[l.base];
    for (int e = blockIdx.y * 256 + threadIdx.x; e < l.n; e += 256 * gridDim.y) {
        const int S = vals ? (int)vals[l.base + e] : praw[l.k0 + e], bf = before[l.base + e] - b0;
        psrc[l.k0 + (far[l.base + e] ? l.n - 1 - bf : e - bf)] = S;
    }
    if (blockIdx.y == 0 && threadIdx.x == 0) nn[l.T] = l.n - (before[l.base + l.n] - b0);
}

static void huge_lists(const NearCtx& c, bool ordered, const int* poff, const int* praw, const int* huge, int nh, int ne,
                       int* psrc, int* nn, hipStream_t s) {
    const dim3 g(nh, (unsigned)std::max(1, std::min(1024, 8192 / nh)));
    DVec<uint64_t> keys;
    DVec<uint32_t> vals;
    if (ordered) {
        int bits = kActKeyBits;
        while (nh - 1 >> (bits - kActKeyBits)) ++bits;
        keys.resize(ne);
        vals.resize(ne);
        k_huge_keys<<<g, 256, 0, s>>>(c, poff, praw, huge, keys.data(), vals.data());
        SFMM_LAUNCH_CHECK();
        radix_sort_u64(keys.data(), vals.data(), ne, bits, s);
    }
    DVec<int> far, before;
    far.resize(ne);
    before.resize((size_t)ne + 1);
    k_huge_flags<<<g, 256, 0, s>>>(c, poff, praw, huge, vals.data(), far.data());
    SFMM_LAUNCH_CHECK();
    scan_excl_i32(far.data(), before.data(), ne, before.data() + ne, s);
    k_huge_place<<<g, 256, 0, s>>>(poff, praw, huge, vals.data(), far.data(), before.data(), psrc, nn);
    SFMM_LAUNCH_CHECK();
}

void near_lists(const NearCtx& c, bool ordered, const int* tl, int ntl, int np, const int* poff, const int* praw,
                int* psrc, int* nn, bool huge, int* pin, hipStream_t s) {
    if (ntl <= 0 || np <= 0) return;
    DVec<int> queue, qhuge;
    queue.resize(2 * ((size_t)ntl + 1));
    qhuge.resize(2 + 2 * (size_t)std::min(ntl, np / (kOneGroupList + 1)));
    int* qmid = queue.data();
    int* qlong = qmid + ntl + 1;
    zero_runs({qmid, sizeof(int)}, {qlong, sizeof(int)}, {qhuge.data(), 2 * sizeof(int)}, s);
    const unsigned g = nblk(64 * (int64_t)ntl, 256);
    if (ordered) k_near_short<true><<<g, 256, 0, s>>>(c, tl, ntl, poff, praw, psrc, nn, qmid, qhuge.data());
    else k_near_short<false><<<g, 256, 0, s>>>(c, tl, ntl, poff, praw, psrc, nn, qmid, qhuge.data());
    SFMM_LAUNCH_CHECK();
    // at most this many lists hold more than the short kernel takes, and more
    // than kMidList entries
    const int nmid = std::min(ntl, np / (ordered ? kShortRanked + 1 : kShortPlain + 1));
    const int nlong = std::min(ntl, np / (kMidList + 1));
    auto launch = [&](auto mid, auto lng) {
        if (nlong > 0) {
            lng<<<std::min(nlong, 1024), 1024, 0, s>>>(c, poff, praw, psrc, nn, qlong);
            SFMM_LAUNCH_CHECK();
        }
        if (nmid > 0) {
            mid<<<std::min(nmid, 4096), 256, 0, s>>>(c, poff, praw, psrc, nn, qmid);
            SFMM_LAUNCH_CHECK();
        }
    };
    if (ordered) launch(k_near_long<true, 256, kMidList>, k_near_long<true, 1024, kOneGroupList>);
    else launch(k_near_long<false, 256, 1>, k_near_long<false, 1024, 1>);
    if (!huge) return;
    SFMM_HIP(hipMemcpyAsync(pin, qhuge.data(), 2 * sizeof(int), hipMemcpyDeviceToHost, s));
    SFMM_HIP(hipStreamSynchronize(s));
    if (pin[1] > 0) huge_lists(c, ordered, poff, praw, qhuge.data(), pin[1], pin[0], psrc, nn, s);
}

}  // namespace sfmm

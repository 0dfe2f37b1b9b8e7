// Host build of rules that the library's host code and kernels share (the same
// headers, compiled for the CPU) for tests/test_host_rules.py.  Modes:
//   sums   : reads counts (decimal, up to 2^30), prints their total as the
//            scans form it (add_sat over any grouping: one by one, in pairs
//            of halves, in tiles of 256 threads of 16), as unsigned numbers
//   stack  : every state of the list walk's stack in LDS, for its one, four and
//            eight waves: prints the states, those from which a step could
//            leave less than the spare places without being a depth-first
//            one, and the most places that a schedule of splits takes which
//            steers for the largest stack and then goes depth first (per
//            number of waves)
//   actkey : reads "round first place" rows, prints the place that comes back
//            from a list's sort key and whether the rows' keys ascend; then the
//            bits that are left for a list's number above the order's key, and
//            1 if a place of the longest list of one workgroup has room below
//   logtab : prints the entries of the pair loop's table
//   log    : reads x, prints the pair loop's log of x and 1/x
//   logerr : largest and root mean square errors of the pair loop's log (in
//            max(1, |log x|)) and reciprocal (relative), against long double,
//            over 2e6 arguments each uniform in (0, 4), spread over 1e-32 ..
//            4 by their logarithm, and in [0.9, 1.1]
#include "../paper_2210_07021_amd/csrc/common.hpp"
#include "../paper_2210_07021_amd/csrc/expand.hpp"
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <random>
#include <vector>

using namespace sfmm;

static uint32_t halves(const std::vector<int>& v, size_t a, size_t b) {
    if (b - a == 1) return (uint32_t)v[a];
    const size_t m = a + (b - a) / 2;
    return (uint32_t)add_sat((int)halves(v, a, m), (int)halves(v, m, b));
}

static std::vector<int> tiles(const std::vector<int>& v, size_t width) {
    std::vector<int> t((v.size() + width - 1) / width, 0);
    for (size_t i = 0; i < v.size(); ++i) t[i / width] = add_sat(t[i / width], v[i]);
    return t;
}

int main(int argc, char** argv) {
    if (argc < 2) return 2;
    if (!strcmp(argv[1], "sums")) {
        std::vector<int> v;
        long x;
        while (scanf("%ld", &x) == 1) v.push_back((int)x);
        uint32_t one = 0;
        for (int c : v) one = (uint32_t)add_sat((int)one, c);
        std::vector<int> t = v;
        while (t.size() > 1) t = tiles(tiles(t, 16), 256);
        printf("%u %u %u\n", one, halves(v, 0, v.size()), (uint32_t)t[0]);
        return 0;
    }
    if (!strcmp(argv[1], "stack")) {
        for (int nw : {1, 4, 8}) {
            const int step = 64 * nw, stack = 1024 * nw, deepest = 29;
            long states = 0, bad = 0;
            int most = 0;
            for (int size = 0; size <= stack - kGroupSpare; ++size) {
                for (int left : {0, 1, step / 2, step, 1 << 30}) {
                    if (size == 0 && left == 0) continue;  // the walk has ended
                    ++states;
                    const GroupTake t = group_take(size, left, step, stack);
                    const int after = size - t.s + 4 * (t.s + t.i);  // all of them split
                    if (t.s > size || t.i > left || t.s + t.i > step || t.s + t.i < 1) ++bad;
                    if (after > stack - kGroupSpare && !(t.s == 1 && t.i == 0)) ++bad;
                    // from here depth first: one level a step, each item splitting
                    int at = std::max(after, size), lev = 1;
                    for (int sz = after; lev < deepest; ++lev) {
                        const GroupTake d = group_take(sz, 0, step, stack);
                        if (d.s != 1) break;
                        sz += 3;
                        at = std::max(at, sz);
                    }
                    most = std::max(most, at);
                }
            }
            printf("%d %ld %ld %d %d\n", nw, states, bad, most, stack);
        }
        return 0;
    }
    if (!strcmp(argv[1], "actkey")) {
        long r, f, e;
        uint64_t last = 0;
        while (scanf("%ld %ld %ld", &r, &f, &e) == 3) {
            const uint64_t k = act_order_key((int)r, (int)f) << kActPlaceBits | (uint64_t)e;
            printf("%d %d\n", (int)(k & ((1u << kActPlaceBits) - 1)), k > last ? 1 : 0);
            last = k;
        }
        printf("%d %d\n", 64 - kActKeyBits, kOneGroupList <= 1 << kActPlaceBits ? 1 : 0);
        return 0;
    }
    if (!strcmp(argv[1], "logtab")) {
        for (int j = 0; j < kLogTab; ++j) printf("%a %a\n", log_tab_entry(j).x, log_tab_entry(j).y);
        return 0;
    }
    if (!strcmp(argv[1], "log")) {
        double2 tab[kLogTab];
        for (int j = 0; j < kLogTab; ++j) tab[j] = log_tab_entry(j);
        double x, lg, inv;
        while (scanf("%lf", &x) == 1) {
            log_recip_tab(x, tab, kLogPoly, &lg, &inv);
            printf("%a %a\n", lg, inv);
        }
        return 0;
    }
    if (!strcmp(argv[1], "logerr")) {
        double2 tab[kLogTab];
        for (int j = 0; j < kLogTab; ++j) tab[j] = log_tab_entry(j);
        std::mt19937_64 g(20221007);
        std::uniform_real_distribution<double> U(0.0, 1.0);
        for (int dom = 0; dom < 3; ++dom) {
            double ml = 0, sl = 0, mi = 0, si = 0;
            const int n = 2000000;
            for (int k = 0; k < n; ++k) {
                const double u = U(g);
                const double x = dom == 0 ? 4.0 * u : dom == 1 ? std::pow(10.0, -32.0 + 32.6 * u) : 0.9 + 0.2 * u;
                if (!(x > 0.0)) continue;
                double lg, inv;
                log_recip_tab(x, tab, kLogPoly, &lg, &inv);
                const long double L = logl((long double)x), I = 1.0L / (long double)x;
                const double el = std::fabs((double)(lg - L)) / std::max(1.0, std::fabs((double)L));
                const double ei = std::fabs((double)((inv - I) / I));
                ml = std::max(ml, el);
                mi = std::max(mi, ei);
                sl += el * el;
                si += ei * ei;
            }
            printf("%.4e %.4e %.4e %.4e\n", ml, std::sqrt(sl / n), mi, std::sqrt(si / n));
        }
        return 0;
    }
    return 2;
}

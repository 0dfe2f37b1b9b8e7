// Host build of rules that the library's host code and kernels share (the same
// headers, compiled for the CPU) for tests/test_host_rules.py.  Modes:
//   sums   : reads counts (decimal, up to 2^30), prints their total as the
//            scans form it (add_sat over any grouping: one by one, in pairs
//            of halves, in tiles of 256 threads of 16), as unsigned numbers
#include "../paper_2210_07021_amd/csrc/common.hpp"
#include <cstdio>
#include <cstring>
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
    return 2;
}

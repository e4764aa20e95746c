// CPU check of the column keys by which the offset-table products and the H-matrix look offsets up
// (plan_key in paper_2105_08798_amd/csrc/plan.h), built with the undefined-behaviour sanitizer by
// tests/test_plan_keys.py.  Input as for plan_check.cpp; the columns of every cell are moved, all by
// the same vector, to places whose keys need more than 32 bits, and every (pad, interface) pair has to
// reach the offset that 64-bit arithmetic finds.  Prints "ok" and returns 0, or the first failure and 1.
#include <cstdio>
#include <vector>

#include "plan.h"

int main(int argc, char** argv) {
    FILE* fp = argc == 2 ? std::fopen(argv[1], "rb") : nullptr;
    if (!fp) return 2;
    auto rd = [&](int32_t* p, size_t n) { return std::fread(p, 4, n, fp) == n; };
    int32_t n_sets = 0;
    if (!rd(&n_sets, 1)) return 2;
    for (int s = 0; s < n_sets; ++s) {
        int32_t n_cells = 0;
        if (!rd(&n_cells, 1)) return 2;
        std::vector<std::vector<int32_t>> ci(n_cells), cb(n_cells);
        for (int c = 0; c < n_cells; ++c) {
            int32_t n[2];
            if (!rd(n, 2)) return 2;
            ci[c].resize(2 * (size_t)n[0]);
            cb[c].resize(2 * (size_t)n[1]);
            if (!rd(ci[c].data(), ci[c].size()) || !rd(cb[c].data(), cb[c].size())) return 2;
        }
        const int32_t far[4][2] = {{0, 0}, {300000000, -400000000}, {-2147000000, 5}, {2147000000, 2147000000}};
        for (const auto& v : far) {
            std::vector<std::vector<int32_t>> fi = ci, fb = cb;
            std::vector<PlanGeom> g;
            for (int c = 0; c < n_cells; ++c) {
                for (size_t k = 0; k < fi[c].size(); ++k) fi[c][k] += v[k & 1];
                for (size_t k = 0; k < fb[c].size(); ++k) fb[c][k] += v[k & 1];
                g.push_back(PlanGeom{(int)fi[c].size() / 2, (int)fb[c].size() / 2, fi[c].data(), fb[c].data()});
            }
            const PlanOffsets o = plan_offsets(g);
            const uint32_t k0 = plan_key(o.d1min, o.d2min, o.w2);
            for (int c = 0; c < n_cells; ++c)
                for (int b = 0; b < g[c].n_b; ++b)
                    for (int i = 0; i < g[c].n_i; ++i) {
                        const int32_t *pb = &fb[c][2 * b], *pi = &fi[c][2 * i];
                        const uint32_t at = plan_key(pb[0], pb[1], o.w2) - k0 - plan_key(pi[0], pi[1], o.w2);
                        const int64_t want = ((int64_t)pb[0] - pi[0] - o.d1min) * o.w2 + ((int64_t)pb[1] - pi[1] - o.d2min);
                        if ((int64_t)at != want || o.lut[at] < 0) {
                            std::fprintf(stderr, "FAIL set %d cell %d pair (%d, %d): place %u, %lld\n", s, c, b, i, at,
                                         (long long)want);
                            return 1;
                        }
                    }
        }
    }
    std::puts("ok");
    return 0;
}

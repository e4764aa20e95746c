// CPU check of the order in which offset-table products take columns (plan_order in
// paper_2105_08798_amd/csrc/plan.cpp), built with the address and undefined-behaviour sanitizers by
// tests/test_column_order.py.  Input as for plan_check.cpp, one cell per set, and per set which of its
// two column sets has to be reordered (bit 0 interface, bit 1 pad) after the cells.  Checks: an order is
// a permutation; it is there exactly where it has to be; consecutive columns lie closer in it; and moving
// the cell far away changes nothing.  Prints "ok" and returns 0, or the first failure and 1.
#include <cmath>
#include <cstdio>
#include <vector>

#include "plan.h"

static double mean_step(const std::vector<int32_t>& c, const std::vector<int32_t>& ord) {
    double s = 0.0;
    const int n = (int)c.size() / 2;
    for (int k = 1; k < n; ++k) {
        const int a = ord.empty() ? k : ord[k], b = ord.empty() ? k - 1 : ord[k - 1];
        s += plan_pair_rho(c[2 * a], c[2 * a + 1], c[2 * b], c[2 * b + 1]) / (n - 1);
    }
    return s;
}

int main(int argc, char** argv) {
    FILE* fp = argc == 2 ? std::fopen(argv[1], "rb") : nullptr;
    if (!fp) return 2;
    auto rd = [&](int32_t* p, size_t n) { return std::fread(p, 4, n, fp) == n; };
    int32_t n_sets = 0, head[3], want = 0;
    if (!rd(&n_sets, 1)) return 2;
    for (int s = 0; s < n_sets; ++s) {
        if (!rd(head, 3) || head[0] != 1) return 2;
        std::vector<int32_t> ci(2 * (size_t)head[1]), cb(2 * (size_t)head[2]);
        if (!rd(ci.data(), ci.size()) || !rd(cb.data(), cb.size()) || !rd(&want, 1)) return 2;
        std::vector<int32_t> oi, ob, fi, fb;
        plan_order(PlanGeom{head[1], head[2], ci.data(), cb.data()}, oi, ob);
        const int got = (oi.empty() ? 0 : 1) | (ob.empty() ? 0 : 2);
        if (got != want) {
            std::fprintf(stderr, "FAIL set %d: reordered %d, expected %d\n", s, got, want);
            return 1;
        }
        for (int k = 0; k < 2; ++k) {
            const std::vector<int32_t>&o = k ? ob : oi, &c = k ? cb : ci;
            if (o.empty()) continue;
            std::vector<int> seen(c.size() / 2, 0);
            for (int32_t x : o)
                if (x < 0 || x >= (int32_t)seen.size() || seen[x]++) {
                    std::fprintf(stderr, "FAIL set %d: not a permutation\n", s);
                    return 1;
                }
            if (o.size() != seen.size() || mean_step(c, o) >= mean_step(c, {})) {
                std::fprintf(stderr, "FAIL set %d: order no closer\n", s);
                return 1;
            }
        }
        for (size_t k = 0; k < ci.size(); ++k) ci[k] += (k & 1) ? -400000000 : 300000000;
        for (size_t k = 0; k < cb.size(); ++k) cb[k] += (k & 1) ? -400000000 : 300000000;
        plan_order(PlanGeom{head[1], head[2], ci.data(), cb.data()}, fi, fb);
        if (fi != oi || fb != ob) {
            std::fprintf(stderr, "FAIL set %d: another order far away\n", s);
            return 1;
        }
    }
    std::puts("ok");
    return 0;
}

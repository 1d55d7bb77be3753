// plan_checks.cpp -- checks of the planner (csrc/plan.cpp) beside those of
// host_checks.cpp; built with g++ and run by tests/test_plan_wide.py.
//
//   plan_checks wide  -- which plans may walk on wide words: at the edge of the
//                        energies' range, by shape, and for whom
#include <algorithm>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <string>
#include <vector>

#include "plan.h"

static int g_fail = 0;
#define CHECK(cond)                                                                \
    do {                                                                           \
        if (!(cond)) {                                                             \
            std::fprintf(stderr, "%s:%d: check failed: %s\n", __FILE__, __LINE__, #cond); \
            if (++g_fail > 20) std::exit(1);                                       \
        }                                                                          \
    } while (0)

using Matrix = std::vector<int32_t>;

// Extremes of E_s(s) + sum_v x_v M[v][s] over all columns s and prefixes x, from
// the definition (Q upper triangular).
static void extremes(const Matrix &Q, int n, int A, int64_t *lo, int64_t *hi)
{
    const int B = n - A;
    *lo = INT64_MAX;
    *hi = INT64_MIN;
    for (int s = 0; s < (1 << B); s++) {
        auto on = [&](int i) { return ((s >> (n - 1 - i)) & 1) != 0; };
        int64_t e = 0, neg = 0, pos = 0;
        for (int i = A; i < n; i++)
            for (int j = i; j < n; j++)
                if (on(i) && on(j)) e += Q[size_t(i) * n + j];
        for (int v = 0; v < A; v++) {
            int64_t m = 0;
            for (int j = A; j < n; j++)
                if (on(j)) m += Q[size_t(v) * n + j];
            (m < 0 ? neg : pos) += m;
        }
        *lo = std::min(*lo, e + neg);
        *hi = std::max(*hi, e + pos);
    }
}

// Random small entries, and one prefix variable's coupling with one suffix
// variable that brings hi - lo to `span` exactly.
static Matrix spanning(int n, int64_t span, int small, uint32_t seed)
{
    std::mt19937 rng(seed);
    const int A = n - 10;
    Matrix Q(size_t(n) * n, 0);
    for (int i = 0; i < n; i++)
        for (int j = i; j < n; j++)
            Q[size_t(i) * n + j] = int32_t(rng() % uint32_t(2 * small + 1)) - small;
    int32_t &big = Q[size_t(3) * n + (n - 7)];
    big = int32_t(-span / 2);
    for (int it = 0; it < 4; it++) {
        int64_t lo, hi;
        extremes(Q, n, A, &lo, &hi);
        big -= int32_t(span - (hi - lo));
    }
    int64_t lo, hi;
    extremes(Q, n, A, &lo, &hi);
    CHECK(hi - lo == span);
    return Q;
}

static qplan::Plan plan(const Matrix &Q, int n, const qubo_options_t *opt = nullptr, bool many = false)
{
    qplan::Plan P;
    std::string msg;
    CHECK(qplan::make_plan(Q.data(), n, QUBO_INT32, opt, &P, &msg, many) == QUBO_OK);
    return P;
}

static int run_wide()
{
    const int64_t edge = int64_t(1) << 21;
    for (uint32_t seed = 0; seed < 4; seed++)
        for (int64_t span : {int64_t(70000), edge / 2, edge - 2, edge - 1, edge, edge + 1, 2 * edge}) {
            const int n = 30 + int(seed);
            const Matrix Q = spanning(n, span, seed == 0 ? 0 : 3 * int(seed), seed);
            const qplan::Plan P = plan(Q, n);
            CHECK(P.tier == 2 && P.mcols == 16 && P.vgpr_levels == 4 && P.A == n - 10);
            int64_t lo, hi;
            extremes(Q, n, P.A, &lo, &hi);
            CHECK(P.pack_shift == -lo);
            CHECK(P.wide == (span <= edge - 1));
            // a batch's and the server's instances, and the other row caches, never
            CHECK(!plan(Q, n, nullptr, true).wide);
            for (int G : {3, 5, 6, 8, 12}) {
                qubo_options_t o{};
                o.vgpr_levels = G;
                CHECK(!plan(Q, n, &o).wide);
            }
        }
    // too few prefix bits
    CHECK(plan(spanning(29, 70000, 2, 9), 29).A == 19 && !plan(spanning(29, 70000, 2, 9), 29).wide);
    // float32
    std::vector<float> F(40 * 40, 0.5f);
    qplan::Plan P;
    std::string msg;
    CHECK(qplan::make_plan(F.data(), 40, QUBO_FP32, nullptr, &P, &msg) == QUBO_OK && !P.wide);
    return 0;
}

int main(int argc, char **argv)
{
    const std::string what = argc > 1 ? argv[1] : "";
    if (what == "wide") run_wide();
    else return 2;
    std::printf("%s: %s\n", what.c_str(), g_fail ? "FAILED" : "ok");
    return g_fail ? 1 : 0;
}

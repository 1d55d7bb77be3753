// serve_checks.cpp -- checks of the serving policy (csrc/serve_policy.cpp) beside
// those of host_checks.cpp; built with g++ and run by tests/test_serve_policy.py.
//
//   serve_checks items  -- the length of a request's work items
//   serve_checks blocks -- the kept memory blocks that are given back
#include <algorithm>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <string>
#include <vector>

#include "serve_policy.h"

static int g_fail = 0;
#define CHECK(cond)                                                                \
    do {                                                                           \
        if (!(cond)) {                                                             \
            std::fprintf(stderr, "%s:%d: check failed: %s\n", __FILE__, __LINE__, #cond); \
            if (++g_fail > 20) std::exit(1);                                       \
        }                                                                          \
    } while (0)

static int run_items()
{
    for (int A = 6; A <= 54; A++) {
        const int L = qsched::item_log(A);
        CHECK(L >= 6 && L <= A);
        // a request that arrives in a tick waits for the items that run: no
        // longer ones than 2^12 steps, unless they would be more than 2^20
        CHECK(L <= 12 || A - L == 20);
        CHECK(A - L <= 20);
        if (A <= 28) CHECK(L <= 10);
        if (A >= 17) CHECK(A - L >= 11);
        CHECK(qsched::longest_item_log(A) >= L);
        CHECK(qsched::longest_item_log(A) <= 12 || A - qsched::longest_item_log(A) == 20);
    }
    return 0;
}

static int run_blocks()
{
    std::mt19937 rng(1);
    for (int rep = 0; rep < 4000; rep++) {
        std::vector<size_t> sizes(rng() % 9);
        size_t total = 0;
        for (size_t &b : sizes) total += b = 1 + rng() % 40;
        std::sort(sizes.begin(), sizes.end());
        const size_t need = rng() % 80;
        const std::vector<size_t> at = qsched::blocks_to_free(sizes, need);
        std::vector<bool> used(sizes.size(), false);
        size_t freed = 0, least = SIZE_MAX;
        for (size_t k : at) {
            CHECK(k < sizes.size() && !used[k]);
            used[k] = true;
            freed += sizes[k];
            least = std::min(least, sizes[k]);
        }
        CHECK(freed >= std::min(need, total));
        if (need == 0) CHECK(at.empty());
        // none of them could have stayed, and no smaller number would do
        if (!at.empty() && total >= need) CHECK(freed - least < need);
        size_t most = 0;
        for (size_t k = 0; k + 1 < at.size(); k++) most += sizes[sizes.size() - 1 - k];
        if (!at.empty() && total >= need) CHECK(most < need);
    }
    return 0;
}

int main(int argc, char **argv)
{
    const std::string what = argc > 1 ? argv[1] : "";
    if (what == "items") run_items();
    else if (what == "blocks") run_blocks();
    else return 2;
    std::printf("%s: %s\n", what.c_str(), g_fail ? "FAILED" : "ok");
    return g_fail ? 1 : 0;
}

// serve_checks.cpp -- checks of the serving policy (csrc/serve_policy.cpp) beside
// those of host_checks.cpp; built with g++ and run by tests/test_serve_policy.py.
//
//   serve_checks items  -- the length of a request's work items
#include <cstdio>
#include <cstdlib>
#include <string>

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

int main(int argc, char **argv)
{
    const std::string what = argc > 1 ? argv[1] : "";
    if (what == "items") run_items();
    else return 2;
    std::printf("%s: %s\n", what.c_str(), g_fail ? "FAILED" : "ok");
    return g_fail ? 1 : 0;
}

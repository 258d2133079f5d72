// Host checks of bz_plan.hpp: what is decided from shapes and options alone.
#include <cstdio>
#include <cstdlib>

#include "bz_plan.hpp"

using namespace bz;

#define CHECK(x)                                                         \
    do {                                                                 \
        if (!(x)) {                                                      \
            std::printf("FAIL %s:%d: %s\n", __FILE__, __LINE__, #x);     \
            std::exit(1);                                                \
        }                                                                \
    } while (0)

// the kernel without tables is dealt to the workgroups that it was measured with
static void check_groups() {
    const int f3[] = {5, 5, 4, 4}, f7[] = {4, 3, 2, 2};
    for (int W = 1; W <= 4; W++) CHECK(prefix_groups(3, W) == f3[W - 1] && prefix_groups(7, W) == f7[W - 1]);
}

static u64 BINOM[65 * 65];
constexpr u64 NO_LIMIT = 1ull << 44;
static bool plain_triples(int p, int n, int k, bool no_term, u64 limit) {
    const int W = (n - k + 31) / 32;
    return triples_worth(p, k, n - k, expected_sets(n, k), expected_rounds(p, n, k, no_term, limit, BINOM),
                         sweep_cap_for(p, W, table_sweep_ops(p)), TRIPLE_LAUNCH_TILES, BINOM);
}

// Rounds that a call can run at all: none past its work limit, all of them
// without termination; triple tables are built for the rounds that run.
static void check_rounds() {
    for (int p : {3, 7})
        for (int n = 2; n <= BZ_MAX_N; n++)
            for (int k = 1; k < n && k <= BZ_MAX_K; k++) {
                const int d = expected_distance(p, n, k);
                CHECK(d >= 1 && d <= n - k + 1 && d == expected_distance(p, n, k));
                const int g = expected_rounds(p, n, k, false, NO_LIMIT, BINOM);
                CHECK(g >= 1 && g <= k && g <= expected_rounds(p, n, k, true, NO_LIMIT, BINOM));
                for (u64 limit : {0ull, 1000ull, 1000000ull, 1ull << 40})
                    for (bool nt : {false, true}) {
                        const int last = expected_rounds(p, n, k, nt, limit, BINOM);
                        // the first stage of round `last` fits the limit behind the rounds before it
                        u64 cum = 0;
                        for (int r = 1; r < last; r++) cum = sat_add(cum, sat_mul(round_codewords(p, k, r, BINOM), expected_sets(n, k)));
                        if (last > 0) CHECK(sat_add(cum, round_codewords(p, k, last, BINOM)) <= limit);
                        if (last < (nt ? k : 1)) {
                            if (last > 0) cum = sat_add(cum, sat_mul(round_codewords(p, k, last, BINOM), expected_sets(n, k)));
                            CHECK(sat_add(cum, round_codewords(p, k, last + 1, BINOM)) > limit);
                        }
                        if (last < TRIPLE_G) CHECK(!plain_triples(p, n, k, nt, limit));
                    }
            }
    CHECK(plain_triples(7, 56, 28, false, NO_LIMIT) && !plain_triples(7, 56, 28, false, 1000000));
    CHECK(plain_triples(3, 80, 28, false, NO_LIMIT) && !plain_triples(3, 80, 28, false, 1000000));
    // a spectrum runs its large rounds, however early the bound would have ended it
    CHECK(!plain_triples(7, 40, 14, false, NO_LIMIT) && plain_triples(7, 40, 14, true, NO_LIMIT));
}

int main() {
    fill_binomials(BINOM);
    check_groups();
    std::printf("OK groups\n");
    check_rounds();
    std::printf("OK rounds\n");
    return 0;
}

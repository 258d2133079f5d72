// Host checks of bz_plan.hpp: what is decided from shapes and options alone.
#include <cstdio>
#include <cstdlib>
#include <random>

#include "bz_plan.hpp"

using namespace bz;

#define CHECK(x)                                                         \
    do {                                                                 \
        if (!(x)) {                                                      \
            std::printf("FAIL %s:%d: %s\n", __FILE__, __LINE__, #x);     \
            std::exit(1);                                                \
        }                                                                \
    } while (0)

static u64 BINOM[65 * 65];
constexpr u64 NO_LIMIT = 1ull << 44;

// the kernel without tables is dealt to the workgroups that it was measured with
static void check_groups() {
    const int f3[] = {5, 5, 4, 4}, f7[] = {4, 3, 2, 2};
    for (int W = 1; W <= 4; W++) {
        CHECK(prefix_groups(3, W, false, 0) == f3[W - 1] && prefix_groups(7, W, false, 0) == f7[W - 1]);
        CHECK(prefix_groups(3, W, true, 100000000) == f3[W - 1] && prefix_groups(3, W, true, 300000000) == 3);
        CHECK(prefix_groups(3, W, true, 0) == (W <= 2 ? 3 : 4) && prefix_groups(7, W, true, 0) == f7[W - 1]);
    }
    // 3^k - 1 over 2 combinations per set
    CHECK(spectrum_size(3, 28, 14, NO_LIMIT, BINOM) == 4782968 && spectrum_size(3, 28, 14, 1000, BINOM) == 1000);
}

static bool plain_triples(int p, int n, int k, bool no_term, u64 limit) {
    const int W = (n - k + 31) / 32;
    const int last = expected_rounds(p, n, k, no_term, limit, BINOM);
    return triples_worth(p, k, n - k, expected_sets(n, k), last, sweep_cap_for(p, W, table_sweep_ops(p)),
                         triple_launch_tiles(p, n, k, no_term, last), BINOM);
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

static bool tables(int p, int n, int k, bool hist = false, bool no_term = false, u64 limit = NO_LIMIT) {
    return tables_by_default(p, n, k, (n - k + 31) / 32 < 1 ? 1 : (n - k + 31) / 32, hist, no_term, false, limit, BINOM);
}

// The expected work against the stages written out, and the shapes on both
// sides of each line of tables_by_default.
static void check_tables() {
    for (int p : {3, 7})
        for (int n = 2; n <= BZ_MAX_N; n += 3)
            for (int k = 1; k < n && k <= BZ_MAX_K; k++) {
                const int m = expected_sets(n, k), d = expected_distance(p, n, k);
                for (int t = 0; t < 6; t++) {
                    const u64 limit = t % 3 == 0 ? 1000 : t % 3 == 1 ? 1000000 : NO_LIMIT;
                    const bool by_round = t >= 3;
                    u64 cum = 0, want = 0;
                    bool end = false;
                    for (int g = 1; g <= k && !end; g++)
                        for (int j = 1; j <= m && !end; j++) {
                            const u64 cw = round_codewords(p, k, g, BINOM);
                            if (sat_add(cum, cw) > limit) {
                                end = true;
                                break;
                            }
                            cum += cw;
                            if (g >= 4) want += cw;
                            int L = 0;
                            for (int i = 1; i <= m; i++) L += bound_c(i <= j ? g : g - 1, k, i <= n / k ? k : n % k);
                            end = L >= d && (j == m || !by_round);
                        }
                    CHECK(expected_work(p, n, k, by_round, limit, BINOM) == want);
                    // no round 4 within the limit: nothing to build tables for
                    if (expected_rounds(p, n, k, true, limit, BINOM) < 4) CHECK(!tables(p, n, k, false, false, limit));
                }
            }
    CHECK(!tables(3, 26, 13) && tables(3, 28, 14) && !tables(3, 84, 14) && tables(3, 90, 20) && !tables(3, 28, 14, true));
    CHECK(!tables(7, 18, 9) && tables(7, 20, 10) && !tables(7, 36, 12) && tables(7, 39, 13) && !tables(7, 45, 13) &&
          tables(7, 66, 12) && !tables(7, 72, 12) && !tables(7, 110, 10) && tables(7, 93, 11) && !tables(7, 24, 3) &&
          tables(7, 16, 5) && !tables(7, 96, 8) && tables(7, 20, 8, true) && !tables(7, 72, 8, true));
    CHECK(!tables(7, 18, 9, false, true) && tables(7, 27, 9, true, true) && !tables(3, 28, 14, false, true) &&
          tables(3, 42, 14, false, true));
    CHECK(tables(7, 56, 28) && !tables(7, 56, 28, false, false, 1000000) && !tables(3, 80, 40, false, false, 100000));
}

// Tables of a batch: side by side, triples only within the budget; an
// allocation that fails with them is tried without.
static void check_layout() {
    std::mt19937 rng(5);
    for (int t = 0; t < 200; t++) {
        std::vector<BatchCode> codes(1 + rng() % 40);
        std::vector<char> want(codes.size());
        const int flags = rng() % 2 ? FLAG_SKIP : 0;
        for (size_t i = 0; i < codes.size(); i++) {
            BatchCode &b = codes[i];
            b.p = rng() % 2 ? 3 : 7;
            b.k = 1 + (int)(rng() % 30);
            b.n = b.k + (int)(rng() % 60);
            b.flags = flags;
            want[i] = triples_fit(b.p, b.k, processed_columns(b.n, b.k, flags != 0));
        }
        for (u64 budget : {(u64)0, (u64)1 << 16, (u64)1 << 20, BATCH_TABLES}) {
            const u64 words = lay_out_tables(codes, want, budget);
            u64 at = 0;
            bool any = false;
            for (size_t i = 0; i < codes.size(); i++) {
                const BatchCode &b = codes[i];
                const int nsym = processed_columns(b.n, b.k, flags != 0);
                CHECK(b.pair_offset == at && (b.triple_off == 0 || (want[i] && at + b.pair_stride * (u64)pair_sets(b.n, b.k) <= budget)));
                CHECK(b.pair_stride == unit_table_size(b.p, b.k, nsym) + (b.triple_off ? triple_table_size(b.p, b.k, nsym) : 0));
                at += b.pair_stride * (u64)pair_sets(b.n, b.k);
                any |= b.triple_off != 0;
            }
            CHECK(at == words && (budget > 0 || !any));
        }
    }
    int calls = 0;
    u64 got = 0;
    auto lay_out = [](u64 budget) { return 100 + budget; };
    auto grow = [&](u64 room) {
        return [&, room](u64 words) {
            calls++;
            got = words;
            return words <= room ? (int)BZ_OK : (int)BZ_ERR_NOMEM;
        };
    };
    CHECK(fit_tables(50, lay_out, grow(150)) == BZ_OK && calls == 1 && got == 150);
    CHECK(fit_tables(50, lay_out, grow(149)) == BZ_OK && calls == 3 && got == 100);
    CHECK(fit_tables(50, lay_out, grow(99)) == BZ_ERR_NOMEM && calls == 5);
    CHECK(fit_tables(0, lay_out, grow(99)) == BZ_ERR_NOMEM && calls == 6);
    CHECK(fit_tables(50, lay_out, [](u64) { return (int)BZ_ERR_DEVICE; }) == BZ_ERR_DEVICE);
    // a server's space: bounded, of the free memory too, and none rather than less than one code's
    const u64 one = max_table_size(128, 1, true, false), plenty = 1ull << 38;
    CHECK(server_triples(1, 128, 1, plenty) == one && server_triples(1024, 128, 1, plenty) * 16 == 3ull << 30);
    CHECK(server_triples(65536, 128, 1, plenty) == SERVER_TRIPLES && server_triples(1024, 128, 1, 8ull << 30) * 16 == 1ull << 30);
    CHECK(server_triples(1024, 128, 1, one * 16 * 7) == 0 && server_triples(1024, 128, 1, 0) == 0);
}

// Ranges handed out never overlap, and one is found whenever a gap holds it.
static void check_arena() {
    std::mt19937 rng(6);
    TableArena a;
    u64 at = 0;
    a.reset(0, 4);
    CHECK(!a.take(1, &at));
    for (u64 size : {10ull, 1000ull}) {
        a.reset(size, 64);
        CHECK(!a.take(size + 1, &at) && !a.take(0, &at) && a.take(size, &at) && at == 0 && !a.take(1, &at));
        a.give(0);
        std::vector<char> map(size, 0);
        std::vector<std::pair<u64, u64>> held;
        for (int t = 0; t < 4000; t++) {
            if (!held.empty() && rng() % 2) {
                const size_t i = rng() % held.size();
                a.give(held[i].first);
                for (u64 w = 0; w < held[i].second; w++) map[held[i].first + w] = 0;
                held.erase(held.begin() + (long)i);
                continue;
            }
            const u64 want = 1 + rng() % (size / 4);
            u64 run = 0, best = 0;
            for (char c : map) best = std::max(best, run = c ? 0 : run + 1);
            const bool ok = a.take(want, &at);
            CHECK(ok == (best >= want));
            if (!ok) continue;
            for (u64 w = at; w < at + want; w++) {
                CHECK(w < size && !map[w]);
                map[w] = 1;
            }
            held.push_back({at, want});
        }
    }
}

int main() {
    fill_binomials(BINOM);
    check_groups();
    std::printf("OK groups\n");
    check_rounds();
    std::printf("OK rounds\n");
    check_tables();
    std::printf("OK tables\n");
    check_layout();
    std::printf("OK layout\n");
    check_arena();
    std::printf("OK arena\n");
    return 0;
}

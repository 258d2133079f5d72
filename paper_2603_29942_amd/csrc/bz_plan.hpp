// bz_plan.hpp -- what the host decides before a launch, from shapes and options
// alone (no device calls, so that it is checked on the CPU).
#pragma once
#include <algorithm>
#include <array>
#include <atomic>
#include <cmath>
#include <stdint.h>
#include <vector>

#include "bz_units.hpp"

namespace bz {

// Workgroups per compute unit of the kernel without tables, at most.  Its
// registers allow one more over F_7, but a wider grid lets more stages start
// at once, whose work is thrown away when an earlier one ends the run (F_7
// without tables, [48, 12] 66.8 us with three, 89.0 with four; [66, 11] 81.4
// and 92.0; [108, 9], four words, 131.1 with two, 136.6 with three).
// With histograms over F_3, three measured better in the runs of up to two
// words that end early ([24, 16] 112 us with five, 88 with three; of three words
// [114, 19] took 174 with four, 219 with three) and in spectra of more than
// 2 10^8 combinations ([54, 18] 4622 and 3815, while [30, 15] took 424 and 447).
// spectrum: its combinations, 0 for a run that ends early.
inline int prefix_groups(int p, int W, bool hist, u64 spectrum) {
    if (p == 3 && hist && (spectrum ? spectrum > 200000000 : W <= 2)) return 3;
    return p == 3 ? (W <= 2 ? 5 : 4) : W == 1 ? 4 : W == 2 ? 3 : 2;
}

// What a plain call's round table depends on (fill_round_table, take_triples):
// p, k, words per plane, the grid of the schedule, tables, triples.  The length
// is no part of it, so calls on codes of many lengths share one.
typedef std::array<int, 6> RoundKey;

// the columns processed per combination
inline int processed_columns(int n, int k, bool skip) { return skip ? n - k : n; }

// 16-byte words between the tables of two sets of a code: the pair table and,
// with triples, the triple table behind it
inline u64 set_table_size(int p, int k, int nsym, bool triples) {
    return unit_table_size(p, k, nsym) + (triples ? triple_table_size(p, k, nsym) : 0);
}
// of every set a code can produce (slots 0 .. pair_sets - 1), plus, on the
// plain path, the slot pair_sets that the workgroup computing the second set
// ahead builds its table in
inline u64 code_table_size(int p, int n, int k, int nsym, bool triples, bool ahead_slot) {
    return (u64)(pair_sets(n, k) + (ahead_slot ? 1 : 0)) * set_table_size(p, k, nsym, triples);
}
// Triples only where a set's table is at most an XCD's L2 (4 MB): every
// wavefront streams it again for each of its tasks.
inline bool triples_fit(int p, int k, int nsym) { return k >= TRIPLE_G && triple_table_size(p, k, nsym) * 16 <= (4u << 20); }

// the largest code_table_size of any code with n <= max_n (with the identity
// skip when skip is 1, without it when 0, either when -1)
inline u64 max_table_size(int max_n, int skip, bool triples, bool ahead_slot) {
    u64 best = 0;
    for (int p : {3, 7})
        for (int n = 1; n <= max_n; n++)
            for (int k = 1; k <= n && k <= BZ_MAX_K; k++)
                for (int sk = 0; sk < 2; sk++) {
                    const int nsym = processed_columns(n, k, sk != 0);
                    if (skip < 0 || skip == sk)
                        best = std::max(best, code_table_size(p, n, k, nsym, triples && triples_fit(p, k, nsym), ahead_slot));
                }
    return best;
}

// ---- memory for tables
// What a batch's tables or a server's triples may take at most, in 16-byte
// words (24 GiB, 4 GiB), and of the device's free memory: the rest of the
// program has uses for it too, and every code runs with pair tables alone.
constexpr u64 BATCH_TABLES = (24ull << 30) / 16, SERVER_TRIPLES = (4ull << 30) / 16;
constexpr u64 FREE_SHARE = 8;
inline u64 table_budget(u64 most, u64 free_bytes) { return std::min(most, free_bytes / FREE_SHARE / 16); }

// Lays out the tables of a batch (offset, stride, triple offset of each code)
// and returns their size.  want[i]: code i takes triples, as long as the tables
// up to its own fit the budget.
inline u64 lay_out_tables(std::vector<BatchCode> &codes, const std::vector<char> &want, u64 budget) {
    u64 words = 0;
    for (size_t i = 0; i < codes.size(); i++) {
        BatchCode &b = codes[i];
        const int nsym = processed_columns(b.n, b.k, (b.flags & FLAG_SKIP) != 0);
        const bool triples = want[i] && words + code_table_size(b.p, b.n, b.k, nsym, true, false) <= budget;
        b.triple_off = triples ? (uint32_t)unit_table_size(b.p, b.k, nsym) : 0u;
        b.pair_stride = (uint32_t)set_table_size(b.p, b.k, nsym, triples);
        b.pair_offset = words;
        words += code_table_size(b.p, b.n, b.k, nsym, triples, false);
    }
    return words;
}
// Allocates what `lay_out(budget)` needs through `grow`, without triples (a
// budget of 0) where that much cannot be had.
template <typename LayOut, typename Grow>
int fit_tables(u64 budget, LayOut &&lay_out, Grow &&grow) {
    const u64 words = lay_out(budget);
    const int st = grow(words);
    if (st != BZ_ERR_NOMEM) return st;
    const u64 least = lay_out((u64)0);
    return least < words ? grow(least) : st;
}

// Ranges of one buffer, first fit: a server's space for the tables of the codes
// that take triples.
class TableArena {
    struct Range {
        u64 at, size;
    };
    std::vector<Range> used;  // by address
    u64 size = 0;

public:
    void reset(u64 words, size_t most_ranges) {
        size = words;
        used.clear();
        used.reserve(most_ranges);
    }
    bool take(u64 words, u64 *at) {
        u64 from = 0;
        size_t i = 0;
        while (i < used.size() && used[i].at - from < words) {
            from = used[i].at + used[i].size;
            i++;
        }
        if (words == 0 || words > size || from > size - words) return false;
        used.insert(used.begin() + (long)i, Range{from, words});
        *at = from;
        return true;
    }
    void give(u64 at) {
        for (size_t i = 0; i < used.size(); i++)
            if (used[i].at == at) {
                used.erase(used.begin() + (long)i);
                return;
            }
    }
};
// Words of that space: 3 MiB a slot (of requests of rate 1/2 with up to 40 rows,
// 28 over F_7, one in two takes 2.8 MB on average, one in four 0.35 MB), and at least
// one code of any kind.
inline u64 server_triples(int slots, int max_n, int skip, u64 free_bytes) {
    const u64 want = std::max((u64)slots * (3u << 20) / 16, max_table_size(max_n, skip, true, false));
    const u64 words = std::min(want, table_budget(SERVER_TRIPLES, free_bytes));
    return words < max_table_size(max_n, skip, true, false) ? 0 : words;
}

// The minimum weight that a random [n, k] code is expected to have: about the
// least d with p^(n-k) words within distance d.  Looked up by the shape after
// the first call for it.
inline int expected_distance(int p, int n, int k) {
    static std::atomic<int16_t> known[2][BZ_MAX_N + 1][BZ_MAX_K + 1];  // 0: not computed yet
    std::atomic<int16_t> &memo = known[p == 7][n][k];
    if (const int d = memo.load(std::memory_order_relaxed)) return d;
    const double goal = (n - k) * std::log((double)p) + std::log((double)(p - 1));
    double lc = 0, sum = 0;  // ln of C(n, d) (p-1)^d, and of their sum
    int d = 0;
    while (d < n && (d == 0 || sum < goal)) {
        d++;
        lc += std::log((double)(n - d + 1) / d * (p - 1));
        sum = d == 1 ? lc : std::max(sum, lc) + std::log1p(std::exp(-std::fabs(sum - lc)));
    }
    d = std::min(d, n - k + 1);
    memo.store((int16_t)d, std::memory_order_relaxed);
    return d;
}
// information sets of a random code
inline int expected_sets(int n, int k) { return n / k + (n % k != 0); }

// Combinations of a run without termination, within the work limit.
inline u64 spectrum_size(int p, int n, int k, u64 max_codewords, const u64 *binom) {
    u64 sum = 0;
    for (int g = 1; g <= k; g++) sum = sat_add(sum, sat_mul(round_codewords(p, k, g, binom), (u64)expected_sets(n, k)));
    return std::min(sum, max_codewords);
}
// The last round that a call on a random [n, k] code is expected to run: the
// one whose bound reaches the expected distance (round g raises it to about
// (g + 1) n / k), or every round without termination, and none past the work
// limit, where the schedule ends.  Only used to decide which tables are worth
// building.
inline int expected_rounds(int p, int n, int k, bool no_term, u64 max_codewords, const u64 *binom) {
    int last = k;
    if (!no_term) last = std::min(std::max((expected_distance(p, n, k) * k + n - 1) / n - 1, 1), k);
    const u64 sets = (u64)expected_sets(n, k);
    u64 cum = 0;
    for (int g = 1; g <= last; g++) {
        if (max_codewords == ~0ull) break;
        const u64 cw = round_codewords(p, k, g, binom);
        if (sat_add(cum, cw) > max_codewords) return g - 1;  // not even its first stage
        cum = sat_add(cum, sat_mul(cw, sets));
    }
    return last;
}
// Combinations of the rounds g >= 4 (those that tables serve) that a call on a
// random [n, k] code is expected to evaluate within its work limit: stage by
// stage until L_{g,j}, tested after every stage or every round, reaches the
// expected distance.
inline u64 expected_work(int p, int n, int k, bool by_round, u64 max_codewords, const u64 *binom) {
    const int d = expected_distance(p, n, k), full = n / k, rest = n % k;
    u64 cum = 0, work = 0;
    for (int g = 1; g <= k; g++) {
        const u64 cw = round_codewords(p, k, g, binom);
        const int sets = expected_sets(n, k);
        for (int j = 1; j <= sets; j++) {
            cum = sat_add(cum, cw);
            if (cum > max_codewords) return work;
            if (g > SUBSET_G) work = sat_add(work, cw);
            const int in = std::min(j, full);
            const int L = full * g + in + (rest ? std::max(0, (j > full ? g + 1 : g) - (k - rest)) : 0);
            if (L >= d && (j == sets || !by_round)) return work;
        }
    }
    return work;
}
// Whether plain calls take pair tables by default: where the rounds from 4 on
// make up for building one per set.  A run that ends before those rounds has
// them among the stages that start at once, so two or three sets of enough rows
// take them whatever the expected work.  Without -> with, in us:
// F_3  k = 12 30.2 -> 30.2 and 35.8 -> 37.0 (two and three sets), 13 40.3 ->
//      42.4; 14 41.1 -> 38.2 and 49.2 -> 45.6, 16 49.9 -> 40.4; of more words
//      by the work: [84, 14] 68.9 -> 76.5, [85, 19] 77.3 -> 79.7 (10^7),
//      [90, 20] 115 -> 89.  With histograms without (they count every sum in
//      LDS either way: [45, 15] ending early 91 -> 116).
// F_7  two sets: k = 9 40.3 -> 46.6, 10 48.5 -> 43.5, 12 49.1 -> 46.1; three:
//      11 and 12 the same, 13 76.7 -> 68.3; else by the work: [72, 12] 98.8 ->
//      124 and [45, 13] 69.5 -> 82.0 (3.5 10^7), [66, 12] 143 -> 126 (5 10^7);
//      of three words and more [110, 10] 155 -> 189 (1.2 10^7), [128, 10]
//      264 -> 224 (2 10^7), [93, 11] 253 -> 155.
//      Up to eight rows in up to four sets: within 3 us of 30 to 45 either way,
//      and with histograms the same (k = 8); the tables of old stay there.
// Spectra (no termination), F_7: [24, 8] 46.9 -> 49.7, [18, 9] 56.2 -> 62.2,
//      [27, 9] 96.6 -> 87.5, [36, 9] 130 -> 73, [20, 10] 175 -> 74; F_3:
//      [28, 14] 122 -> 130, [42, 14] 192 -> 72, [30, 15] 209 -> 135.
inline bool tables_by_default(int p, int n, int k, int W, bool hist, bool no_term, bool by_round, u64 max_codewords,
                              const u64 *binom) {
    if (p == 3 && (hist || k < 14)) return false;
    // the schedule has a round 4 at all
    const int sets = expected_sets(n, k);
    u64 cum = 0;
    for (int g = 1; g <= SUBSET_G; g++) cum = sat_add(cum, sat_mul(round_codewords(p, k, g, binom), (u64)sets));
    if (k <= SUBSET_G || sat_add(cum, round_codewords(p, k, SUBSET_G + 1, binom)) > max_codewords) return false;
    if (no_term) return k > (p == 3 ? 14 : 9) || (k == (p == 3 ? 14 : 9) && sets >= 3);
    if (p == 3 && W <= 2) return true;
    if (p == 7 && k <= 8) return sets <= 4 && (k == 8 || !hist);
    if (p == 7 && ((k >= 10 && sets <= 2) || (k >= 13 && sets == 3))) return true;
    const u64 work = expected_work(p, n, k, by_round, max_codewords, binom);
    return work >= (p == 3 ? 10000000u : W <= 2 ? 40000000u : 18000000u);
}
// Triple tables pay when the rounds up to `last` save more tiles than the
// tables take to build (a unit costs about 200 VALU instructions, a tile of 64
// bases 100: one tile per 32 units) and, on the plain path, than their launch
// takes.
// (batches of 512 with a work limit of 10^6, which ends them in round 4: 750 us
// without triples, 1324 us with triples chosen as if they ran on)
inline bool triples_worth(int p, int k, int nsym, int sets, int last, uint32_t cap, u64 launch_tiles, const u64 *binom) {
    if (last < TRIPLE_G || !triples_fit(p, k, nsym)) return false;
    u64 build = sat_mul(triple_tiles(p, k, -1), (u64)sets) + launch_tiles, saved = 0;
    for (int g = TRIPLE_G; g <= last && round_combos(p, g) < (1ull << 32); g++) {
        u64 c3;
        triple_round(p, k, g, cap, false, binom, &c3);
        const u64 c2 = pair_round_cost(p, k, g, cap, binom);
        if (c2 > c3) saved = sat_add(saved, sat_mul(c2 - c3, (u64)sets));
    }
    return saved > build;
}
// The launch in tiles, 8 us of them; fewer for a run that its limit ends, which
// has no stage beyond that starts at once and is thrown away (limits of 2 10^8:
// [84, 14] over F_7 206 -> 155 us, [120, 30] over F_3 116 -> 101).
inline u64 triple_launch_tiles(int p, int n, int k, bool no_term, int last) {
    return last < expected_rounds(p, n, k, no_term, ~0ull, nullptr) ? 15000 : 40000;
}

}  // namespace bz

// Host-side checks of the pair tables as matrix operands (bz_units.hpp), built
// with g++: the FP4 values that the device multiplies are decoded here and
// summed in double.
//
//   weights  for both fields, every table layout and word count: the sums of
//            the products of random vectors give the weight of x + h y for
//            every multiplier h, and the first bound of F_7 is no smaller than
//            any of a rotation's two agreement counts
//   order    the units of the rows of a block are one range, the pairs of the
//            rows s >= s_lo are the first ones, and each unit's pair is the
//            one its index says; the same for the triples
//   triples  the rounds that take them: every base meets the triples above its
//            top row, their combinations add up to the round's, the blocks of a
//            group abut, and take_triples keeps tasks and flags together
//   reports  the plain kernel's rules replayed (first tile, claims, deals): the
//            tiles and workgroups of each copy are the ones it counts on
//
// Prints "OK <check>" per passing check; exits 1 on the first failure.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <random>
#include <set>
#include <utility>
#include <vector>

#include "bz_units.hpp"

using namespace bz;

#define CHECK(c)                                                    \
    do {                                                            \
        if (!(c)) {                                                 \
            std::printf("FAIL %s:%d %s\n", __FILE__, __LINE__, #c); \
            std::exit(1);                                           \
        }                                                           \
    } while (0)

static std::mt19937_64 rng(7);

static double fp4(u32 nib) {
    static const double v[8] = {0, 0.5, 1, 1.5, 2, 3, 4, 6};
    return (nib & 8 ? -1.0 : 1.0) * v[nib & 7];
}
// one lane's 32 products of two operand words (registers r = 0 .. 3)
static double dot(const u32 (&a)[4], const u32 (&b)[4]) {
    double s = 0;
    for (int r = 0; r < 4; r++)
        for (int i = 0; i < 8; i++) s += fp4((a[r] >> (4 * i)) & 15) * fp4((b[r] >> (4 * i)) & 15);
    return s;
}
template <int P, int W>
static int symbol(const u32 (&x)[3][W], int t) {
    int v = 0;
    for (int b = 0; b < 3; b++) v |= (int)((x[b][t / 32] >> (t % 32)) & 1u) << b;
    return v;
}
template <int P, int W>
static void draw(u32 (&x)[3][W], int n, int zeros) {
    std::memset(x, 0, sizeof x);
    for (int t = 0; t < n; t++) {
        const int v = (int)(rng() % 10) < zeros ? 0 : (int)(rng() % P);
        for (int b = 0; b < 3; b++) x[b][t / 32] |= (u32)((v >> b) & 1) << (t % 32);
    }
}
template <int P, int W>
static int weight(const u32 (&x)[3][W], const u32 (&y)[3][W], int h, int n) {
    int w = 0;
    for (int t = 0; t < n; t++) w += (symbol<P, W>(x, t) + h * symbol<P, W>(y, t)) % P != 0;
    return w;
}

template <int P, int W, int SCH>
static void check_weights(int n) {
    constexpr int NP = unit_pieces(SCH, W), REC = unit_rec_words(SCH, W);
    CHECK(unit_scheme(P, n) == SCH);
    for (int it = 0; it < 40; it++) {
        u32 x[3][W], y[3][W];
        draw<P, W>(x, n, it % 4 * 2);
        draw<P, W>(y, n, it % 3 * 3);
        if (it % 5 == 4) std::memcpy(x, y, sizeof x);
        u32 pl[NP][2], nz[NP][2], sg[NP][2], rec[2][REC];
        base_slots<P, W, SCH>(x, pl, nz, sg);
        unit_record<P, W, SCH>(y, 0, rec[0]);
        unit_record<P, W, SCH>(y, 1, rec[1]);
        int wx = 0;
        for (int t = 0; t < n; t++) wx += symbol<P, W>(x, t) != 0;
        if (P == 3) {
            double c = 0, e = 0, o = 0;
            for (int i = 0; i < NP; i++)
                for (int h = 0; h < 2; h++) {
                    u32 ae[4], ao[4], be[4], bo[4], kb[4];
                    for (int r = 0; r < 4; r++) {
                        ae[r] = fp4_unit(rec[h][2 * i], r);
                        ao[r] = ae[r] | fp4_signs(rec[h][2 * i + 1], r);
                        be[r] = fp4_nonzero3(nz[i][h], r);
                        bo[r] = fp4_one(nz[i][h], r) | fp4_signs(sg[i][h], r);
                        kb[r] = fp4_minus2(r);
                    }
                    c += dot(ae, kb);
                    e += dot(ae, be);
                    o += dot(ao, bo);
                }
            const int wm = weight<P, W>(x, y, P - 1, n), wp = weight<P, W>(x, y, 1, n);
            CHECK(2 * wx - (c + e + o) == 2 * wm);
            CHECK(2 * wx - (c + e - o) == 2 * wp);
        } else {
            for (int t = 0; t < 3; t++) {
                double cb = 0, b = 0, c = 0, d = 0, o = 0;
                for (int i = 0; i < NP; i++)
                    for (int h = 0; h < 2; h++) {
                        u32 a0[4], a[4], ao[4], bb[4], bf[4], bo[4], kb[4], kf[4];
                        for (int r = 0; r < 4; r++) {
                            a0[r] = fp4_unit(rec[h][unit_word(SCH, 0, i)], r);
                            a[r] = fp4_unit(rec[h][unit_word(SCH, t, i)], r);
                            ao[r] = a[r] | fp4_signs(rec[h][unit_sign_word(SCH, i)], r);
                            bb[r] = fp4_bound(nz[i][h], pl[i][h], r);
                            bf[r] = fp4_matched(nz[i][h], pl[i][h], r);
                            bo[r] = fp4_one(pl[i][h], r) | fp4_signs(sg[i][h], r);
                            kb[r] = slot_used(SCH, i, h) ? fp4_minus1(r) : 0u;
                            kf[r] = slot_used(SCH, i, h) ? fp4_minus2(r) : 0u;
                        }
                        cb += dot(a0, kb);
                        c += dot(a0, kf);
                        b += dot(a, bb);
                        d += dot(a, bf);
                        o += dot(ao, bo);
                    }
                const int wm = weight<P, W>(x, y, (7 - (1 << t)) % 7, n), wp = weight<P, W>(x, y, 1 << t, n);
                CHECK(2 * wx - (c + d + o) == 2 * wm);  // x - 2^t y
                CHECK(2 * wx - (c + d - o) == 2 * wp);
                CHECK(wx - (cb + b) <= wm && wx - (cb + b) <= wp);
            }
        }
    }
}

static void check_order() {
    for (int p : {3, 7})
        for (int k = 2; k <= BZ_MAX_K; k++) {
            const int np = k * (k - 1) / 2;
            std::set<std::pair<int, int>> seen;
            for (int s = 0; s < k - 1; s++)
                for (int L = s + 1; L < k; L++) {
                    const int e = (int)pair_first(s, k) + L - s - 1;
                    const int u = first_unit(p, k, e + 1), i = k - 1 - s, j = k - 1 - L;
                    CHECK(u == (i * (i - 1) / 2 + j) * (p - 1));
                    CHECK(first_unit(p, k, e) == u + p - 1);
                    int a, b;
                    pair_of(u / (p - 1), k, &a, &b);
                    CHECK(b == i && a == j);
                    seen.insert({s, L});
                }
            CHECK((int)seen.size() == np && first_unit(p, k, np) == 0);
            CHECK(table_tiles(p, k) * 32 >= (u64)np * (p - 1));
            // the pairs of the rows s >= s_lo are the first units
            for (int s = 0; s < k - 1; s++) CHECK(first_unit(p, k, (int)pair_first(s, k)) == (k - 1 - s) * (k - s) / 2 * (p - 1));
        }
}

static void check_triples() {
    u64 binom[65 * 65];
    fill_binomials(binom);
    for (int p : {3, 7})
        for (int k = TRIPLE_G; k <= BZ_MAX_K; k++) {
            // unit order: colex rank of the reversed rows, prefixes above each row
            int r = 0;
            for (int i = 2; i < k; i++)
                for (int j = 1; j < i; j++)
                    for (int l = 0; l < j; l++, r++) CHECK(r == choose3(i) + choose2(j) + l);
            CHECK(triple_units(p, k, -1) == r * units_per_triple(p));
            for (int q = 0; q < k; q++) {
                int above = 0;
                for (int a = q + 1; a < k; a++) above += choose2(k - 1 - a);
                CHECK(triple_units(p, k, q) == above * units_per_triple(p));
            }
            for (uint32_t cap : {1u, 4u, 35u, 142u, 1846u}) {
                const uint32_t cap3 = triple_cap(p, cap);
                RoundTable t, t0;
                fill_round_table(p, k, 2, 768, 4500, binom, &t0);
                t = t0;
                take_triples(p, k, cap, 768, binom, &t);
                for (int g = TRIPLE_G; g <= k && round_combos(p, g) < (1ull << 32); g++) {
                    u64 tasks[2] = {0, 0}, combos = 0, cost;  // without and with runs
                    for (int q = g - 4; q <= k - 4; q++) {
                        const u64 bases = triple_bases(p, binom[q * 65 + g - 4], round_combos(p, g));
                        const uint32_t tiles = triple_tiles(p, k, q), nb = triple_blocks(tiles, cap3);
                        CHECK(nb >= 1 && triple_block_start(tiles, nb, 0) == 0 && triple_block_start(tiles, nb, nb) == tiles);
                        for (uint32_t b = 0; b < nb; b++) {
                            const uint32_t d = triple_block_start(tiles, nb, b + 1) - triple_block_start(tiles, nb, b);
                            CHECK(d >= 1 && d <= cap3);
                        }
                        for (int r = 0; r < 2; r++) {
                            const uint32_t d = triple_digits(p, g, tiles, nb, bases, r != 0);
                            CHECK(d <= (uint32_t)(g - 4) && d <= max_digits(p) && (r || d == 0));
                            // a run is whole (the lanes' bases end together) and bounded
                            CHECK(bases % run_len(p, d) == 0 || bases == ~0ull);
                            CHECK(d == 0 || run_len(p, d) * ((tiles + nb - 1) / nb) <= RUN_TILES);
                            tasks[r] = sat_add(tasks[r], triple_tasks(p, bases, nb, d));
                        }
                        combos = sat_add(combos, sat_mul(bases, (u64)triple_units(p, k, q) * (u64)(p - 1)));
                    }
                    for (int r = 0; r < 2; r++) CHECK(tasks[r] == triple_round(p, k, g, cap, r != 0, binom, &cost));
                    const u64 want = round_codewords(p, k, g, binom);
                    CHECK(combos == want || want == ~0ull || combos == ~0ull);
                    if (t.vcap[g - 1] & TRIPLES) CHECK(t.tasks[g - 1] == tasks[t.vcap[g - 1] & 1] && g < t.cut_g);
                    else CHECK(t.tasks[g - 1] == t0.tasks[g - 1] && t.vcap[g - 1] == t0.vcap[g - 1]);
                }
                for (int g = 1; g < TRIPLE_G; g++) CHECK(t.tasks[g - 1] == t0.tasks[g - 1]);
            }
        }
}

static void check_reports() {
    for (int round = 0; round < 400; round++) {
        const uint32_t grid = round % 4 == 0 ? 1 + (uint32_t)(rng() % 40) : 32 + (uint32_t)(rng() % 1500);
        const uint32_t deal = grid + (round % 3 ? 0 : (uint32_t)(rng() % 900));
        // a schedule: stages that start at once until the deal grid is full
        StageDesc st[40];
        int ns = 0;
        u64 off = 0;
        for (; ns < 40; ns++) {
            StageDesc &d = st[ns];
            std::memset(&d, 0, sizeof d);
            d.tiles = rng() % 5 == 0 ? 1 + rng() % (40 * deal) : 1 + rng() % 60;
            d.nowait = off < deal;
            d.rot = (uint32_t)((deal - off % deal) % deal);
            off += d.tiles;
        }
        u64 tiles = 0;
        const int sp = pool_stages(st, ns, deal, &tiles);
        const uint32_t C = pool_slices(grid), copies = report_copies(grid);
        CHECK(C % copies == 0);
        std::vector<std::vector<uint32_t>> got(ns, std::vector<uint32_t>(copies, 0));
        for (uint32_t b = 0; b < grid; b++)
            if (b < tiles) got[pool_stage_of(st, sp, 0, b, deal)][b % copies]++;
        for (uint32_t c = 0; c < C; c++)
            for (uint32_t i = 0; grid + pool_tile(c, i, C) < tiles; i++)
                got[pool_stage_of(st, sp, 0, grid + pool_tile(c, i, C), deal)][c % copies]++;
        for (int s = sp; s < ns; s++) {
            st[s].parts = (uint32_t)(st[s].tiles < grid ? st[s].tiles : grid);
            st[s].rot %= grid;
            for (uint32_t b = 0; b < grid; b++)
                if (tile_of(0, b, grid, st[s].rot) < st[s].tiles) got[s][b % copies]++;
        }
        for (int s = 0; s < ns; s++) {
            uint32_t sum = 0;
            for (uint32_t c = 0; c < copies; c++) {
                const uint32_t n = s < sp ? report_pool_tiles((uint32_t)nowait_offset(st[s].rot, deal),
                                                              (uint32_t)st[s].tiles, grid, c, copies)
                                          : report_groups(st[s].rot, st[s].parts, grid, c, copies);
                CHECK(n == got[s][c] && n < 65536);
                sum += n;
            }
            CHECK(sum == (s < sp ? st[s].tiles : st[s].parts));
        }
    }
}

int main() {
    for (int n = 1; n <= 32; n++) check_weights<3, 1, 0>(n);
    for (int n = 33; n <= 64; n++) check_weights<3, 2, 0>(n);
    for (int n = 65; n <= 96; n++) check_weights<3, 3, 0>(n);
    for (int n = 97; n <= 128; n++) check_weights<3, 4, 0>(n);
    for (int n = 1; n <= 21; n++) check_weights<7, 1, 1>(n);
    for (int n = 22; n <= 32; n++) check_weights<7, 1, 2>(n);
    for (int n = 33; n <= 42; n++) check_weights<7, 2, 3>(n);
    for (int n = 43; n <= 64; n++) check_weights<7, 2, 4>(n);
    for (int n = 65; n <= 96; n++) check_weights<7, 3, 5>(n);
    for (int n = 97; n <= 128; n++) check_weights<7, 4, 5>(n);
    std::printf("OK weights\n");
    check_order();
    std::printf("OK order\n");
    check_triples();
    std::printf("OK triples\n");
    check_reports();
    std::printf("OK reports\n");
    return 0;
}

// bz_units.hpp -- the pair tables as matrix-core operands (shared by host and
// device).
//
// Weights as an inner product.  For symbol vectors x (a lane's exact base) and
// y (a unit of the table) over the processed columns, wt(x - y) = n' minus the
// positions where x and y agree, and agreements are inner products of small
// integer vectors that the matrix cores multiply in FP4 with FP32 sums (all
// of them small integers, so each result is exact):
//   F_3  x, y in {0, 1, -1}: with S = sum x^2 y^2 and D = sum x y,
//        wt(x -+ y) = wt(x) + wt(y) - (3 S +- D) / 2.
//   F_7  a nonzero symbol is +-2^e (Sec. 4.2).  With S = the positions where
//        both are nonzero, E_t = those with e_x = e_y + t and O_t = the same
//        sum signed by the two signs,
//        wt(x -+ 2^t y) = wt(x) + wt(y) - S - (E_t +- O_t) / 2.
// One unit so serves p - 1 multiples: 2 over F_3 (the rows of S and D), 6 over
// F_7 (t = 0, 1, 2 and both signs).
//
// Operand layout.  v_mfma_f32_32x32x64_f8f6f4 takes 32 units (A, one per row)
// and 32 bases (B, one per column); lane l holds row or column l % 32 and the
// products k = 32 (l / 32) .. + 31 as eight 4-bit values in each of four
// registers.  The order of the products is free as long as A and B agree, so
// register r, nibble i stands for bit 4 i + r of a 32-bit word and a word
// expands with one `and` per register (fp4_unit).  A "slot" is one such
// word: (piece i, half h) is product range 32 h .. 32 h + 31 of the i-th
// matrix instruction.  Over F_7 a base's slot holds one plane P_e (the symbols
// +-2^e) and the unit multiplied by 2^t has plane P_{e-t} there:
//   scheme 1 (n' <= 21)  one piece: the planes 21 bits apart in 64 bits
//   scheme 2 (n' <= 32)  two pieces: slots P_0, P_1, P_2, unused.  The record's
//                        words X_t = P_{h-t} serve piece 0 as X_t and piece 1
//                        as X_{t+1}: no word is kept twice
//   scheme 3 (n' <= 42)  two pieces: the first 32 columns as in scheme 2, the
//                        fourth slot holds the other 10 columns of all planes
//   scheme 4 (n' <= 64)  three pieces, piece e = P_e; 2^t y is a renaming
//   scheme 5 (n' <= 128) six pieces, piece (e, pair of words)
// and over F_3 scheme 0 has ceil(W / 2) pieces.
#pragma once
#include <stdint.h>

#include "bz_arith.hpp"
#include "bz_state.hpp"

namespace bz {

BZ_HD int unit_scheme(int p, int nsym) { return p == 3 ? 0 : nsym <= 21 ? 1 : nsym <= 32 ? 2 : nsym <= 42 ? 3 : nsym <= 64 ? 4 : 5; }
// matrix instructions per product
constexpr int unit_pieces(int sch, int W) {
    return sch == 0 ? (W + 1) / 2 : sch == 1 ? 1 : sch <= 3 ? 2 : sch == 4 ? 3 : 6;
}
// 32-bit words of a unit that one lane (one half) holds: its planes, then its signs
constexpr int unit_rec_words(int sch, int W) { return sch == 0 ? 2 * ((W + 1) / 2) : sch == 3 || sch == 5 ? 8 : 4; }

// units of a pair table (R_s + c R_L for s < L and every c in F_p^*) and the
// tiles of 32 that hold them
BZ_HD u64 table_tiles(int p, int k) { return ((u64)k * (u64)(k - 1) / 2 * (u64)(p - 1) + 31) / 32; }
// 16-byte words of a pair table over nsym columns: per tile, the records of 64 lanes
BZ_HD u64 unit_table_size(int p, int k, int nsym) {
    const int W = (nsym + 31) / 32 < 1 ? 1 : (nsym + 31) / 32;
    return table_tiles(p, k) * 16 * (u64)unit_rec_words(unit_scheme(p, nsym), W);
}
// The units are stored last pair first, so that the pairs of the rows s >= s_lo
// (which end the row-major order of the pairs) are the first units: unit u
// belongs to the pair s = k-1-i, L = k-1-j with i(i-1)/2 + j = u / (p-1), and
// its coefficient c is u % (p-1) + 1.  The pairs e in [e0, e1) of the row-major
// order are the units [first_unit(e1), first_unit(e0)).
BZ_HD int first_unit(int p, int k, int e) { return (k * (k - 1) / 2 - e) * (p - 1); }

// ---- triples: units of three rows
// A base of g-2 rows meets only the pairs above its top row, k(k-1)/(g(g-1)) of
// them on average (6 to 30 where the time goes): the base's operands then cost
// more than the products.  Rounds g >= 5 can instead give a base g-3 rows and
// sweep the sums of the three highest, R_a + c1 R_b + c2 R_c with a < b < c:
// about (k-2)/(g-2) (p-1) times as many units for each base, from a second
// table per set.  Unit u = r (p-1)^2 + (c1-1)(p-1) + c2-1 of the triple
// a = k-1-i, b = k-1-j, c = k-1-l with colex rank r = C(i,3) + C(j,2) + l of
// l < j < i, so that the triples above row q are again the first ones.
constexpr uint32_t TRIPLES = 1u << 31;  // in StageDesc::vcap of a round that takes triples; + 1: in runs
constexpr int TRIPLE_G = 5;             // the first round that can
BZ_HD int choose2(int n) { return n * (n - 1) / 2; }
BZ_HD int choose3(int n) { return n * (n - 1) / 2 * (n - 2) / 3; }
BZ_HD int units_per_triple(int p) { return (p - 1) * (p - 1); }
// units of the triples above row q, and the tiles that hold them
BZ_HD int triple_units(int p, int k, int q) { return k - 1 - q < 3 ? 0 : choose3(k - 1 - q) * units_per_triple(p); }
BZ_HD uint32_t triple_tiles(int p, int k, int q) { return (uint32_t)(triple_units(p, k, q) + 31) / 32; }
BZ_HD uint32_t pair_tiles(int p, int k, int q) { return (uint32_t)(choose2(k - 1 - q) * (p - 1) + 31) / 32; }
// 16-byte words of a triple table over nsym columns
BZ_HD u64 triple_table_size(int p, int k, int nsym) {
    const int W = (nsym + 31) / 32 < 1 ? 1 : (nsym + 31) / 32;
    return (u64)triple_tiles(p, k, -1) * 16 * (u64)unit_rec_words(unit_scheme(p, nsym), W);
}
// A q-group's tiles are cut into blocks of at most about triple_cap tiles,
// the size of a task in pairs (sweep_cap_for) as tiles; block b starts at tile
// b tiles / blocks.
BZ_HD uint32_t triple_cap(int p, uint32_t cap) { return cap * (uint32_t)(p - 1) / 32 < 1 ? 1u : cap * (uint32_t)(p - 1) / 32; }
BZ_HD uint32_t triple_blocks(uint32_t tiles, uint32_t cap3) { return (tiles + cap3 - 1) / cap3; }
BZ_HD uint32_t triple_block_start(uint32_t tiles, uint32_t nb, uint32_t b) { return (uint32_t)((u64)tiles * b / nb); }
// What a round costs, in tiles of 32 units swept by 64 bases: a sweep's set-up
// (decoding, operands; about 500 VALU instructions against 100 of a tile)
// counts as five.  Round g (>= TRIPLE_G) takes triples where they cost less.
constexpr uint32_t SWEEP_COST = 5;
// pairs: bases of the group with top row q, their blocks of rows s
BZ_HD u64 pair_group_cost(int p, int k, int q, u64 bases, uint32_t nb) {
    return sat_mul(ceil64(bases), (u64)nb * SWEEP_COST + pair_tiles(p, k, q));
}
BZ_HD u64 triple_group_cost(uint32_t tiles, u64 bases, uint32_t nb) {
    return sat_mul(ceil64(bases), (u64)nb * SWEEP_COST + tiles);
}
// the bases of g-3 rows with top row q; M = (p-1)^(g-3), as for pairs
BZ_HD u64 triple_bases(int p, u64 binom_q_g4, u64 M) { return sat_mul(binom_q_g4, M / (u64)(p - 1)); }
// Low coefficient digits of the bases that a lane runs through itself, as with
// pairs (see digits_of): most bases meet few triples, and decoding one takes
// as long as ten tiles, so that a task of short sweeps takes (p-1)^d bases per
// lane, each one row away from the last, up to RUN_TILES tiles in all (a
// batch of 256: 25.7, 24.9 and 23.3 ms with 48, 96 and 192).  [56, 28] over F_7: 3.05 -> 1.96 ms; 128 mixed requests, 34 -> 25 ms.
// runs: the round has enough tasks for it (runs_pay).
constexpr uint32_t RUN_TILES = 192;
BZ_HD uint32_t triple_digits(int p, int g, uint32_t tiles, uint32_t nb, u64 bases, bool runs) {
    const uint32_t fit = runs ? RUN_TILES / ((tiles + nb - 1) / nb) : 0;  // (every group has a tile)
    if (fit < (uint32_t)(p - 1)) return 0;
    uint32_t d = p == 3 ? 31u - (uint32_t)__builtin_clz(fit) : 1u;
    const uint32_t most = (uint32_t)(g - 4) < max_digits(p) ? (uint32_t)(g - 4) : max_digits(p);
    d = d < most ? d : most;
    const uint32_t b = digits_by_bases(p, bases);
    return b < d ? b : d;
}
BZ_HD u64 triple_tasks(int p, u64 bases, uint32_t nb, uint32_t vd) {
    return sat_mul(ceil64(p == 3 ? bases >> vd : (vd ? bases / (u64)(p - 1) : bases)), nb);
}
// tasks (64 lanes by one block) and cost of round g with triples
BZ_HD u64 triple_round(int p, int k, int g, uint32_t cap, bool runs, const u64 *binom, u64 *cost) {
    const uint32_t cap3 = triple_cap(p, cap);
    const u64 M = round_combos(p, g);
    u64 tasks = 0;
    *cost = 0;
    for (int q = g - 4; q <= k - 4; q++) {
        const u64 bases = triple_bases(p, binom[q * 65 + (g - 4)], M);
        const uint32_t tiles = triple_tiles(p, k, q), nb = triple_blocks(tiles, cap3);
        tasks = sat_add(tasks, triple_tasks(p, bases, nb, triple_digits(p, g, tiles, nb, bases, runs)));
        *cost = sat_add(*cost, triple_group_cost(tiles, bases, nb));
    }
    return tasks;
}
BZ_HD u64 pair_round_cost(int p, int k, int g, uint32_t cap, const u64 *binom) {
    const u64 M = round_combos(p, g);
    u64 cost = 0;
    for (int q = g - 3; q <= k - 3; q++)
        cost = sat_add(cost, pair_group_cost(p, k, q, sat_mul(binom[q * 65 + (g - 3)], M), qgroup_blocks(k, cap, q)));
    return cost;
}
// A round table whose rounds take triples where they cost less, in runs where
// a stage then still has a tile for every workgroup of the grid.
BZ_HD void take_triples(int p, int k, uint32_t cap, uint32_t grid, const u64 *binom, RoundTable *t) {
    for (int g = TRIPLE_G; g <= k; g++) {
        if (round_combos(p, g) >= (1ull << 32) || g >= t->cut_g) break;
        u64 c3;
        const u64 tasks = triple_round(p, k, g, cap, false, binom, &c3);
        if (c3 >= pair_round_cost(p, k, g, cap, binom)) continue;
        const u64 tv = triple_round(p, k, g, cap, true, binom, &c3);
        const bool runs = runs_pay(tv, grid);
        t->tasks[g - 1] = runs ? tv : tasks;
        t->vcap[g - 1] = TRIPLES | (runs ? 1u : 0u);
    }
}

// F_7: one-hot planes of the exponents and the sign plane (symbol = -2^e)
BZ_HD void f7_exponents(u32 b0, u32 b1, u32 b2, u32 (&pl)[3], u32 &sgn) {
    sgn = (b0 & b1) | (b0 & b2) | (b1 & b2);  // 6, 5, 3: the complements of 1, 2, 4
    pl[0] = b0 ^ sgn;
    pl[1] = b1 ^ sgn;
    pl[2] = b2 ^ sgn;
}

// three 21-bit planes in 64 bits, the low or the high word
BZ_HD u32 pack21(u32 a, u32 b, u32 c, int half) { return half ? (b >> 11) | (c << 10) : a | (b << 21); }

// The record of a unit with planes y for the lanes of one half.
template <int P, int W, int SCH>
BZ_HD void unit_record(const u32 (&y)[3][W], int half, u32 (&rec)[unit_rec_words(SCH, W)]) {
    if constexpr (P == 3) {
        for (int i = 0; i < unit_pieces(0, W); i++) {
            const int w1 = 2 * i + 1 < W ? 2 * i + 1 : 2 * i;
            const bool in = half == 0 || 2 * i + 1 < W;
            const u32 a = half ? y[0][w1] : y[0][2 * i], b = half ? y[1][w1] : y[1][2 * i];
            rec[2 * i] = in ? a | b : 0u;
            rec[2 * i + 1] = in ? b : 0u;
        }
    } else {
        u32 pl[W][3], sg[W];
        for (int w = 0; w < W; w++) f7_exponents(y[0][w], y[1][w], y[2][w], pl[w], sg[w]);
        if constexpr (SCH == 1) {
            for (int t = 0; t < 3; t++) rec[t] = pack21(pl[0][(3 - t) % 3], pl[0][(4 - t) % 3], pl[0][(5 - t) % 3], half);
            rec[3] = pack21(sg[0], sg[0], sg[0], half);
        } else if constexpr (SCH == 2 || SCH == 3) {
            for (int t = 0; t < 3; t++) rec[t] = half ? pl[0][(4 - t) % 3] : pl[0][(3 - t) % 3];
            rec[3] = sg[0];
            if constexpr (SCH == 3) {
                constexpr int V = W - 1;
                for (int t = 0; t < 3; t++)
                    rec[4 + t] = half ? pl[V][(3 - t) % 3] | (pl[V][(4 - t) % 3] << 10) | (pl[V][(5 - t) % 3] << 20)
                                      : pl[0][(5 - t) % 3];
                rec[7] = half ? sg[V] | (sg[V] << 10) | (sg[V] << 20) : sg[0];
            }
        } else if constexpr (SCH == 4) {
            constexpr int V = W > 1 ? 1 : 0;
            for (int e = 0; e < 3; e++) rec[e] = half ? pl[V][e] : pl[0][e];
            rec[3] = half ? sg[V] : sg[0];
        } else {
            for (int i = 0; i < 2; i++) {
                const int w0 = 2 * i < W ? 2 * i : 0, w1 = 2 * i + 1 < W ? 2 * i + 1 : 0;
                const bool in = 2 * i + half < W;
                for (int e = 0; e < 3; e++) rec[2 * e + i] = !in ? 0u : half ? pl[w1][e] : pl[w0][e];
                rec[6 + i] = !in ? 0u : half ? sg[w1] : sg[w0];
            }
        }
    }
}
// The record words that are piece i of the unit times 2^t: its plane and its signs.
constexpr int unit_word(int sch, int t, int i) {
    return sch == 1 ? t : sch == 2 ? (t + i) % 3 : sch == 3 ? (i == 0 ? t : 4 + t) : sch == 4 ? (i - t + 3) % 3
           : 2 * ((i / 2 - t + 3) % 3) + i % 2;
}
constexpr int unit_sign_word(int sch, int i) { return sch == 3 ? 3 + 4 * i : sch == 5 ? 6 + i % 2 : 3; }

// The slots of a base with planes x, per piece and half: over F_3 (nonzero,
// negative), over F_7 (plane, nonzero, sign).  Unused slots are 0.
template <int P, int W, int SCH>
BZ_HD void base_slots(const u32 (&x)[3][W], u32 (&pl)[unit_pieces(SCH, W)][2], u32 (&nz)[unit_pieces(SCH, W)][2],
                      u32 (&sg)[unit_pieces(SCH, W)][2]) {
    constexpr int NP = unit_pieces(SCH, W);
    if constexpr (P == 3) {
        for (int i = 0; i < NP; i++)
            for (int h = 0; h < 2; h++) {
                const bool in = 2 * i + h < W;
                const int w = in ? 2 * i + h : 0;
                pl[i][h] = nz[i][h] = in ? x[0][w] | x[1][w] : 0u;
                sg[i][h] = in ? x[1][w] : 0u;
            }
    } else {
        u32 e[W][3], s[W], n[W];
        for (int w = 0; w < W; w++) {
            f7_exponents(x[0][w], x[1][w], x[2][w], e[w], s[w]);
            n[w] = x[0][w] | x[1][w] | x[2][w];
        }
        if constexpr (SCH == 1) {
            for (int h = 0; h < 2; h++) {
                pl[0][h] = pack21(e[0][0], e[0][1], e[0][2], h);
                nz[0][h] = pack21(n[0], n[0], n[0], h);
                sg[0][h] = pack21(s[0], s[0], s[0], h);
            }
        } else if constexpr (SCH == 2 || SCH == 3) {
            for (int h = 0; h < 2; h++) {
                pl[0][h] = e[0][h];
                nz[0][h] = n[0];
                sg[0][h] = s[0];
            }
            pl[1][0] = e[0][2];
            nz[1][0] = n[0];
            sg[1][0] = s[0];
            if constexpr (SCH == 3) {
                constexpr int V = W - 1;
                pl[1][1] = e[V][0] | (e[V][1] << 10) | (e[V][2] << 20);
                nz[1][1] = n[V] | (n[V] << 10) | (n[V] << 20);
                sg[1][1] = s[V] | (s[V] << 10) | (s[V] << 20);
            } else {
                pl[1][1] = nz[1][1] = sg[1][1] = 0u;
            }
        } else {
            for (int i = 0; i < NP; i++)
                for (int h = 0; h < 2; h++) {
                    const int q = SCH == 4 ? i : i / 2, wi = SCH == 4 ? h : 2 * (i % 2) + h;
                    const bool in = wi < W;
                    const int w = in ? wi : 0;
                    pl[i][h] = in ? e[w][q] : 0u;
                    nz[i][h] = in ? n[w] : 0u;
                    sg[i][h] = in ? s[w] : 0u;
                }
        }
    }
}
// slot (i, h) holds products (else the base's operand is 0 there, and the unit's word may be anything)
constexpr bool slot_used(int sch, int i, int h) { return !(sch == 2 && i == 1 && h == 1); }

// ---- expanding words to FP4 registers
// bit 4 i + r of w to bit `at` of nibble i.  FP4 codes: bit 3 the sign; 1 is
// 0.5, 2: 1, 3: 1.5, 4: 2, 5: 3, 6: 4, 7: 6.
BZ_HD u32 fp4_bits(u32 w, int r, int at) {
    return (at >= r ? w << (at - r) : w >> (r - at)) & (0x11111111u << at);
}
// A unit's word keeps its bits where they are: registers 0, 1, 2 take one
// `and` and hold 0.5, 1, 2; register 3, shifted by one, holds 2.  A base's
// registers carry the inverse factors 4, 2, 1, 1, so that every product of a
// set bit and a base value v is 2 v.
BZ_HD u32 fp4_unit(u32 w, int r) { return (r == 3 ? w >> 1 : w) & (0x11111111u << (r == 3 ? 2 : r)); }
// the signs of a word
BZ_HD u32 fp4_signs(u32 w, int r) { return fp4_bits(w, r, 3); }
// F_3: 1.5 where n is set (products 3)
BZ_HD u32 fp4_nonzero3(u32 n, int r) {
    return r == 0 ? fp4_bits(n, 0, 0) * 7u : r == 1 ? fp4_bits(n, 1, 0) * 5u : fp4_bits(n, r, 0) * 3u;
}
// 0.5 where w is set (products 1)
BZ_HD u32 fp4_one(u32 w, int r) { return fp4_bits(w, r, r == 0 ? 2 : r == 1 ? 1 : 0); }
// F_7 bound: 0.5 where n is set, 1 where p (within n) is (products 1 and 2)
BZ_HD u32 fp4_bound(u32 n, u32 p, int r) {
    return r == 0   ? fp4_bits(n, 0, 2) | fp4_bits(p, 0, 1)
           : r == 1 ? fp4_bits(n ^ p, 1, 1) | fp4_bits(p, 1, 2)
                    : fp4_bits(n ^ p, r, 0) | fp4_bits(p, r, 1);
}
// F_7 signed sums: 1 where n is set, 1.5 where p is (products 2 and 3)
BZ_HD u32 fp4_matched(u32 n, u32 p, int r) {
    return r == 0   ? fp4_bits(n, 0, 1) * 3u | fp4_bits(p, 0, 0)
           : r == 1 ? fp4_bits(n, 1, 2) | fp4_bits(p, 1, 0)
                    : fp4_bits(n, r, 1) | fp4_bits(p, r, 0);
}
// constants: products -1 (v = -0.5) and -2
BZ_HD u32 fp4_minus1(int r) { return r == 0 ? 0xCCCCCCCCu : r == 1 ? 0xAAAAAAAAu : 0x99999999u; }
BZ_HD u32 fp4_minus2(int r) { return r == 0 ? 0xEEEEEEEEu : r == 1 ? 0xCCCCCCCCu : 0xAAAAAAAAu; }

}  // namespace bz

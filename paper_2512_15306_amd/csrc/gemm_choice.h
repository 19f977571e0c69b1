// Host side of the contractions: which kernel a problem takes.  Plain functions of the sizes, without a kernel in sight.
#pragma once
#include <math.h>
#include <stdint.h>
#include <stdlib.h>

#include "llmq_kernels.h"

namespace llmq {

constexpr int BK = 128;                                     // contraction bytes of a K step
constexpr int kXcds = 8;
constexpr int kNoEdge = 0, kEdge = 1, kEdgeUnaligned = 2;    // kinds of the tile kernel (gemm_tile.h)

// Whether the LDS of a CU holds one workgroup of the two-stage tile kernel: two fit of up to six units, 80 KB each.
constexpr bool alone_on_cu(int ni, int nj) { return ni * nj > 6; }

// Workgroups of the tile kernel that run on the chip at once (a multiple of the XCD count), as the models of time below count them: two to a CU of
// 128 x 128 tiles, one of all others.  (Two of 192 x 128 and 128 x 192 fit as well, but counted that way their measured times are fitted worse: see tile_us.)
// LLMQ_GEMM_SLOTS overrides it for tests, so that small problems meet the many-rounds code paths.
inline int resident_slots(int num_cus, int ni, int nj) {
    if (const char* e = tuning_env("LLMQ_GEMM_SLOTS")) { const int v = atoi(e); if (v >= kXcds && v % kXcds == 0) return v; }
    return (num_cus / kXcds) * kXcds * ((ni == 2 && nj == 2) ? 2 : 1);
}

struct TileChoice {
    int ni, nj;       // 0, 0: no tuned tile divides the problem
};

struct EdgeChoice {
    int ni, nj;       // 0, 0: the generic kernel
    int edge;         // kEdge or kEdgeUnaligned
};

// Whether the generic kernel finishes first.  Its waves of 16 x 16 outputs (BF16: lanes of one output) have no LDS to fill
// and no tile to write out, which makes it the faster one for small problems, as long as its operands can be loaded in
// vectors or the contraction is one K step long.  FP8: the same sums, so the same bytes.  A model in microseconds: waits of
// one wave, and for every further round of workgroups per CU; fitted to 1712 shapes in four layouts up to 4001 x 1001 outputs
// and T = 2048 while the tile kernel had four waves; with eight it is 0.2 to 0.4 us faster, and of 6000 shapes two take the generic kernel that are more
// than 3 % faster on a tile of 128 x 128.  Generic / tile kernel (eight waves up to 15 K steps):
//   both operands in rows, R x C x T   100 x 136 x 64 3.3 / 4.6, x 512 4.8 / 5.6, x 1024 6.8 / 6.8, x 2048 10.7 / 9.5;  1000 x 520 x 64 4.4 / 4.9,
//     x 256 6.0 / 5.3, x 384 7.3 / 5.6;  2000 x 1000 x 64 7.9 / 5.4;  T no multiple of 32: 100 x 136 x 400 7.1 / 5.5, x 50 6.9 / 7.3, x 1001 47 / 14
//   C no multiple of 8 (stores of two bytes a lane)   300 x 300 x 64 3.3 / 7.9, x 1024 6.8 / 10.1;  1000 x 1001 x 256 7.6 / 8.5, x 512 11.0 / 9.1
//   B T-major   100 x 136 x 64 6.2 / 6.3, x 256 9.7 / 7.2;  300 x 300 x 50 8.1 / 9.5;   both T-major   300 x 300 x 16 7.1 / 8.8, x 32 9.7 / 9.1
//   BF16   40 x 40 x 25 4.0 / 6.8, x 65 6.5 / 6.9, x 100 9.7 / 7.1;  300 x 300 x 25 5.4 / 9.7, 513 x 520 x 25 10.1 / 7.6;  100 x 136 x 8 3.0 / 4.7, x 16 4.1 / 4.7
inline bool generic_is_faster(int64_t R, int64_t C, int64_t T, bool ta, bool tb, bool accumulate, bool with_amax, bool bf16, int num_cus) {
    if (bf16) {                                                             // (T in bytes)
        const int64_t most = T <= 16 ? 320000 : T % 16 == 0 ? (T <= 32 ? 60000 : 0) : T <= 56 ? 160000 : T <= 104 ? 60000 : T <= 144 ? 52000 : 0;
        return R * C <= most;
    }
    if (R * C > ((int64_t)1 << 23)) return false;
    const double steps = (double)((T + BK - 1) / BK);
    const int64_t workgroups = ((R + 31) / 32) * ((C + 31) / 32);
    const double more = (double)((workgroups + num_cus - 1) / num_cus - 1);
    const bool one = T <= BK, odd_width = C % 8 != 0;
    double generic, tile;
    if (!ta && !tb && T % 16 == 0) {
        generic = (T % 32 == 0 ? 2.5 : 5.4) + 0.5 * steps + more * (0.25 + 0.44 * steps);
        tile = 4.9 + 0.29 * steps;
    } else if (!ta && !tb && one) {
        generic = 6.6 + more * 0.03 * (double)T;
        tile = 7.2;
    } else if (!ta && one) {
        generic = T <= 16 ? 6.3 + more * 0.6 : T % 32 == 0 ? 6.0 + more * 0.8 : 7.9 + more * 0.02 * (double)T;
        tile = T % 16 == 0 && C % 16 == 0 ? 5.0 : 6.5;
    } else if (ta && one) {
        generic = T <= 16 ? 6.7 + more * 0.6 : (C <= 32 ? 7.9 : 9.2) + more * 0.9;
        tile = R % 16 == 0 && C % 16 == 0 ? 5.0 : 6.5;
    } else {
        return false;
    }
    const double rows = R < 16 ? 16.0 : R > 64 ? 64.0 : (double)R;          // that a wave of the tile kernel writes out
    if (odd_width) tile += (rows - 16.0) / 48.0 * 2.1;
    if (accumulate) { generic += 0.9 + 0.68 * more; tile += odd_width ? 1.2 : 0.6; }
    // every wave of the generic kernel raises the same word, and atomics on one address follow each other at 9.5 ns (forward call
    // of 300 x 256 -> 1024, 1216 waves: 25 us with it, 13.5 with the tile kernel)
    if (with_amax) generic += 0.0095 * (double)(((R + 15) / 16) * ((C + 15) / 16));
    return generic < tile + 0.4e-6 * (double)R * (double)C;
}

// Tile and kind of a ragged problem, by the same model with the tiles rounded up.  Against the best of the four tiles of even sides, forced,
// over 28 shapes from 1000^3 to 9000^2 x 1000: 0.7 % behind on average with aligned rows, 2.6 % with unaligned ones and 1.4 % with both
// operands T-major; no other efficiencies of this model do better on the first two.
// Tiles of 192 rows (aligned rows only) stand between the others where those would need another round: without / with them, operands in rows,
// R x C x T 4114 x 4156 x 4784 138.8 / 115.8 us, 4911 x 6786 x 6912 242 / 208, 2385 x 3578 x 2448 47.7 / 40.6, 8026 x 2771 x 6864 194 / 166,
// 5971 x 1623 x 1104 29.0 / 24.7;  B T-major 2385 x 3584 x 2448 35.9 / 30.1;  both T-major 4128 x 4160 x 4784 116 / 96, 4912 x 6800 x 6912
// 246 / 205;  BF16 4114 x 4156 x 2392 131 / 113.  Short contractions of operands in rows lose with 192 x 128
// (3901 x 1149 x 720 14.1 / 14.4), hence the lower figure.  (On some of these the tiles of better_tile below are faster still.)
// Where all 128 x 128 tiles are resident at once, two to a CU, they hide each other's prologue and output, so 192 x 128 needs K steps to win by (least_192).
// 128 x 128 / 192 x 128 time by K steps 1, 2, 3 to 4, 5 to 8, 9 to 16, more, over 1200 shapes: 0.98, 1.01, 1.04, 1.09, 1.09, 1.11;  added to the output
// 0.93, 0.96, 1.02, 1.05, 1.06, 1.09;  widths no multiples of 8 (stores of single elements) 0.91, 0.92, 0.96, 0.98, 1.00, 1.05;  with absmax (fewer
// atomics) 1.12, 1.13, 1.07, 1.03, 1.04, 1.11.  192 x 256 tiles of odd widths lose the same way where there are several rounds of them: 3328 x 10548 x 128 added
// to the output 43.9 / 57.4, 7105 x 4754 x 64 36.1 / 45.7.
inline EdgeChoice choose_edge_tile(int64_t R, int64_t C, int64_t T, int num_cus, bool ta, bool tb, bool slabs_a, bool slabs_b, bool accumulate, bool with_amax, bool bf16) {
    EdgeChoice best{0, 0, 0};
    // 32-bit offsets from the first row of a tile, of operands (as above) and of the output; the guarded loads need 16
    // bytes in every row of an operand
    if (T >= (1ll << 23) || C >= (1ll << 22) || T < 16 || (ta && R < 16) || (tb && C < 16)) return best;
    const bool aligned_a = ta ? R % 16 == 0 : slabs_a || T % 16 == 0, aligned_b = tb ? C % 16 == 0 : slabs_b || T % 16 == 0;
    best.edge = aligned_a && aligned_b ? kEdge : kEdgeUnaligned;
    if (const char* force = tuning_env("LLMQ_GEMM_EDGE_TILE")) {
        const int ni = force[0] - '0', nj = force[0] && force[1] ? force[2] - '0' : 0;
        if ((ni == 2 || ni == 4 || (ni == 3 && best.edge == kEdge)) && (nj == 2 || nj == 4)) { best.ni = ni; best.nj = nj; return best; }
        if (ni == 0) return best;                             // 0x0: the generic kernel
    }
    if (generic_is_faster(R, C, T, ta, tb, accumulate, with_amax, bf16, num_cus)) return best;
    if (best.edge == kEdge && ((R + 127) / 128) * ((C + 127) / 128) <= resident_slots(num_cus, 2, 2) / 2) { best.ni = best.nj = 2; return best; }   // as above
    const int least_192 = C % 8 != 0 ? 17 : with_amax ? 1 : accumulate ? 3 : 2;
    const bool resident = ((R + 127) / 128) * ((C + 127) / 128) <= resident_slots(num_cus, 2, 2);
    double best_cost = 0;
    for (int ni = 4; ni >= 2; --ni)
        for (int nj = 4; nj >= 2; nj -= 2) {
            if (ni == 3 && best.edge != kEdge) continue;
            if (ni == 3 && nj == 2 && resident && (T + BK - 1) / BK < least_192) continue;
            const int64_t tiles = ((R + 64 * ni - 1) / (64 * ni)) * ((C + 64 * nj - 1) / (64 * nj));
            if (tiles > kMaxWorkgroups) continue;
            const int per_cu = (ni == 2 && nj == 2) ? 2 : 1;
            const int64_t slots = resident_slots(num_cus, ni, nj);
            const int64_t rounds = (tiles + slots - 1) / slots;
            const bool odd_rounds = C % 8 != 0 && T <= 8 * BK && rounds > 1;      // (outputs of single elements, round after round)
            const double e = per_cu == 2 ? (T <= 3072 ? 0.90 : 0.80) : ni == 3 ? (nj == 4 ? (odd_rounds ? 0.74 : 0.83) : T <= 1024 && !tb ? 0.68 : 0.74) : (ni == nj ? 1.0 : 0.77);
            const double cost = (double)rounds * per_cu * ni * nj / e;
            if (best.ni == 0 || cost < best_cost * 0.97) { best.ni = ni; best.nj = nj; best_cost = cost; }
        }
    return best;
}

// ---- A second look at problems of many tiles.
//
// A tile and its form: kNoEdge where the tile divides the problem, kEdge where it is guarded (or a large tile adds to the output).
struct TilePlan {
    int ni, nj, edge;           // ni = 0: the generic kernel
    bool shares = false;        // its last round is shared out (choose_split), where scratch is given
};

// Microseconds of a contraction of `tiles` tiles: a launch, then for every round of tiles the prologue and output of a tile and its K steps.  A last
// round that is not full takes less than a full one: under the power cap the CUs that have a tile run faster.  One table for FP8 and BF16 (a step is
// 128 bytes of the contraction in both: steps fitted to BF16 alone differ by 0-2 %, 256 x 320 by 3, and choose no better).  Fitted to 515 (guarded tiles: 380) shapes of 700 to
// 16384 rows and columns and T of 256 to 16384 in all layouts, every tile forced on every shape; the cost of adding to the output and the 128 x 192 tile, of which
// two fit a CU, to 21009 of 64 to 52000: 5 to 10 % root mean square, most of it at T = 256 to 512.  (Tiles of six units counted as two to a CU fit worse: 12 % against 8 for 192 x 128, 13 against 10 for 128 x 192.)
// odd_width: C is no multiple of 8, so the outputs leave element by element; what that adds to a guarded tile of every round (`odd`) is fitted to 8843
// shapes of such widths, 64 x 128 outputs and T = 256 to 16384 and more.  The 256 x 320 tile loses most, by trips of 64 lanes over a wave's 160 columns.
inline double tile_us(const TilePlan& p, int64_t tiles, int64_t steps, bool accumulate, bool odd_width, int64_t slots) {
    struct Fit { int ni, nj; double whole_tile, whole_step, whole_add, guarded_tile, guarded_step, guarded_add, odd; };
    static const Fit fits[] = {{4, 5, 9.5, 1.507, 0, 10.0, 1.532, 6.7, 16.2},  {5, 4, 8.6, 1.500, 0, 9.8, 1.508, 5.2, 13.2},  {4, 4, 7.4, 1.243, 3.0, 8.4, 1.268, 4.2, 10.6},
                               {3, 4, 5.9, 0.984, 2.1, 6.5, 1.009, 2.8, 8.2},  {4, 3, 5.7, 1.009, 2.1, 0, 0, 0, 0},           {3, 3, 4.2, 0.870, 1.4, 0, 0, 0, 0},
                               {4, 2, 4.2, 0.788, 1.4, 4.9, 0.822, 2.1, 5.3},  {2, 4, 4.5, 0.794, 1.1, 4.9, 0.813, 2.1, 5.3}, {3, 2, 2.2, 0.616, 0.8, 2.4, 0.618, 1.4, 2.9},
                               {2, 3, 2.7, 0.660, 0.8, 0, 0, 0, 0},            {2, 2, 3.2, 0.829, 1.2, 3.6, 0.873, 1.4, 3.1}};
    const double rest = (double)(tiles % slots) / (double)slots;
    const double rounds = (double)(tiles / slots) + (rest > 0 ? 0.69 + 0.31 * rest : 0.0);
    for (const Fit& f : fits)
        if (f.ni == p.ni && f.nj == p.nj) {
            const bool guarded = p.edge != kNoEdge;
            return 3.1 + rounds * ((guarded ? f.guarded_tile : f.whole_tile) + (double)steps * (guarded ? f.guarded_step : f.whole_step) +
                                   (accumulate ? (guarded ? f.guarded_add : f.whole_add) : 0.0) + (odd_width ? f.odd * (accumulate ? 1.18 : 1.0) : 0.0));
        }
    return 0.0;
}

// What the models of choose_tile and choose_edge_tile do not weigh: the large tiles 256 x 320 (4 x 5) and 320 x 256 (5 x 4), and guarded tiles of 256 x 256
// and 192 x 256 also where a smaller tile divides the problem.  Returns `base`, their choice, or a tile that tile_us has 2 % or more ahead of it.
//   Large tiles: a tenth fewer operand bytes per product from L2 to LDS and from LDS to registers, which is what the power cap leaves the matrix cores
//   short of, and other counts of tiles.  FP8 4 x 4 / large, microseconds: 16384 x 5120 x 5120 (5 / 4 whole rounds) 295.7 / 288.4;  55296 x 5120 x 16384 3103 /
//   3001;  8192 x 5120 x 13824 (2.5 / 2 rounds) 402 / 360;  4096 x 5120 x 3072 (1.25 / 1 round) 68.0 / 48.9, BF16 (256 x 128 tiles before) 120 / 89;
//   4096 x 2560 x 4096 (one round of either) 40.3 / 47.9.
//   Guarded tiles, 128 x 128 that divide the problem / guarded: 4480 x 2176 x 8320 94.6 / 68.2 (192 x 256), 1792 x 7552 x 4096 60.2 / 49.8 (256 x 256),
//   3584 x 5632 x 7680 142.7 / 109.5 (256 x 320), 4480 x 13184 x 3072 182 / 142 (320 x 256).
//   Widths that are no multiples of 8, the tile before / the one this table takes without `odd` / with it:  8160 x 4982 x 448 52.7 / 63.5 / 52.7 and 768 x 45462 x 384
//   42.9 / 58.5 / 42.9 (128 x 128, 256 x 320, 128 x 128);  8960 x 5812 x 1024 110 / 100 / 100 (256 x 256, 320 x 256).  Over the 8843 shapes 1.7 % faster than without a
//   second look on average, 7 of them more than 3 % slower; without `odd` 1.1 %, and 561 (down to 0.73 times).
//   Short contractions: with one figure per unit of tile for the addition to the output, and 128 x 192 tiles a quarter slower than they are, 3232 x 43520 x 480 added to the
//   output took 256 x 320 tiles (197.1, 256 x 256 170.2) and 12928 x 576 x 384 192 x 256 (13.2, 128 x 192 11.6).
// Over 21009 shapes of widths that are multiples of 8 (7068 of them with T = 256 to 512): 2.7 % faster than without on average (4.6 % from 17 K steps on), 101 of them more than 3 % slower (7 more
// than 10), of which the noise of the timing is a part; 1.1 % behind the best of these tiles.  320 x 192, 192 x 320, 320 x 128 and 128 x 320 tiles would add 0.2 % each.
// scale: what sharing out the last round of `base` saves of its time; shared: whether it is shared out.  Such tiles take their sums in another order than whole ones,
// so which of the two it is does not depend on whether the output is added to.  LLMQ_GEMM_ANY_TILE=IxJ (tests): that tile, guarded if need be; 0: `base`.
inline TilePlan better_tile(int64_t R, int64_t C, int64_t T, int num_cus, bool ta, bool tb, bool slabs_a, bool slabs_b, bool accumulate, const TilePlan& base, double scale, bool shared = false) {
    // 32-bit offsets from the first row of a tile of up to 320; whole 16-byte chunks; A T-major alone has no guarded form
    if ((ta && !tb) || T < 16 || T >= (1ll << 22) || C >= (1ll << 22)) return base;
    if (!(ta ? R % 16 == 0 : slabs_a || T % 16 == 0) || !(tb ? C % 16 == 0 : slabs_b || T % 16 == 0)) return base;
    auto form = [&](int ni, int nj, bool adds) {
        const bool guarded = R % (64 * ni) != 0 || C % (64 * nj) != 0 || T % BK != 0 || (adds && ni * nj > 16);
        return TilePlan{ni, nj, guarded ? kEdge : kNoEdge};
    };
    const char* force = tuning_env("LLMQ_GEMM_ANY_TILE");
    if (force && force[0] >= '2' && force[0] <= '5' && force[1] == 'x') return form(force[0] - '0', force[2] - '0', accumulate);
    if (base.ni == 0 || T < 2 * BK) return base;                          // (the table starts there)
    if (force || tuning_env("LLMQ_GEMM_TILE") || tuning_env("LLMQ_GEMM_EDGE_TILE") || tuning_env("LLMQ_GEMM_SPLIT")) return base;       // (tests of the other tiles)
    const bool priced_add = accumulate && !shared;
    auto us = [&](const TilePlan& p) -> double {
        const int64_t tiles = ((R + 64 * p.ni - 1) / (64 * p.ni)) * ((C + 64 * p.nj - 1) / (64 * p.nj));
        return tiles > kMaxWorkgroups ? 0.0 : tile_us(p, tiles, (T + BK - 1) / BK, priced_add, C % 8 != 0, resident_slots(num_cus, p.ni, p.nj));
    };
    if (((R + 127) / 128) * ((C + 127) / 128) <= resident_slots(num_cus, 2, 2) / 2 && base.ni == 2 && base.nj == 2) return base;       // four LDS stages
    TilePlan best = base;
    double best_us = us(base) * scale * 0.98;
    const int others[4][2] = {{4, 5}, {5, 4}, {4, 4}, {3, 4}};
    for (const auto& o : others) {
        const double t = us(form(o[0], o[1], priced_add));
        if (t > 0.0 && t < best_us) { best = form(o[0], o[1], accumulate); best_us = t; }
    }
    return best;
}

// What the small tiles are compared with, in microseconds: the 128 x 128 tile with four LDS stages, whole or with guarded edges, or the
// generic kernel where that is the faster of the two.
inline double other_tiles_us(int64_t R, int64_t C, int64_t T, bool accumulate, bool with_amax, bool bf16, int num_cus) {
    const double steps = (double)((T + BK - 1) / BK), n = (double)R * (double)C;
    const bool ragged = R % 128 != 0 || C % 128 != 0 || T % BK != 0;
    if (ragged && generic_is_faster(R, C, T, false, false, accumulate, with_amax, bf16, num_cus)) {
        // BF16, outputs x elements of T, generic / 32 x 32: 64 x 8 2.2 / 3.2, 4096 x 8 2.5 / 3.4, 60000 x 8 2.7 / 3.5, 130000 x 8 3.1 / 3.6,
        // 200000 x 8 3.8 / 4.0, 320000 x 8 4.5 / 5.5;  64 x 16 2.9 / 3.2, 1024 x 16 3.6 / 3.4, 60000 x 16 3.8 / 3.5
        if (bf16) return T <= 16 ? 2.3 + 7e-6 * n : n <= 128 ? 2.9 : 3.8;
        const double load = (double)(((R + 31) / 32) * ((C + 31) / 32)) / num_cus, rounds = ceil(load) - 1.0;        // workgroups per CU, on the fullest CU beyond the first
        return 1.75 + 0.4 * steps + load * (0.17 + 0.125 * steps) + rounds * (0.18 + 0.24 * steps) + (T % 32 != 0 ? 2.8 : 0.0) + (C % 8 == 0 ? 0.43 : 0.0) +
               (R >= 32 ? 0.3 : 0.0) + (accumulate ? 0.35 + 0.53 * load : 0.0) + (with_amax ? 0.013 * (double)(((R + 15) / 16) * ((C + 15) / 16)) - 0.35 : 0.0);
    }
    const double tiles = (double)(((R + 127) / 128) * ((C + 127) / 128)), part = (R < 128 ? R / 128.0 : 1.0) * (C < 128 ? C / 128.0 : 1.0);
    const double odd = C % 8 != 0 ? (R < 64 ? R / 64.0 : 1.0) * (C < 64 ? C / 64.0 : 1.0) : 0.0;        // stores of single elements
    return (ragged ? 4.5 + 0.318 * steps : 3.9 + 0.326 * steps) + 0.007 * tiles + odd * (accumulate ? 3.1 : 2.4) + (accumulate ? 0.5 * part : 0.0) +
           (with_amax ? 0.0095 * tiles : 0.0);
}
// The same for tiles of side x side: rounds of them, each with its stages of four K steps and its output
inline double small_tiles_us(int side, int64_t R, int64_t C, int64_t T, bool accumulate, bool with_amax, int num_cus) {
    const double tiles = (double)(((R + side - 1) / side) * ((C + side - 1) / side)), rounds = (double)(((int64_t)tiles + num_cus - 1) / num_cus);
    const double stages = (double)((T + 4 * BK - 1) / (4 * BK)), part = (R < side ? (double)R / side : 1.0) * (C < side ? (double)C / side : 1.0);
    const double odd = C % 4 != 0 ? part : 0.0;
    const double per_round = side == 32 ? 1.25 + 0.41 * stages + (accumulate ? 0.3 * part + 0.8 * odd : 0.2 * odd)
                                        : 1.3 + 0.86 * stages + part * (accumulate ? 1.2 : 0.65) + odd * (accumulate ? 2.8 : 0.6);
    return 1.75 + rounds * per_round + (side == 32 ? 0.44 : 0.77) * tiles / num_cus + (with_amax ? 0.0095 * tiles : 0.0);
}

// The small tiles: their side, or 0 for another kernel.  The models above, fitted to 26000 FP8 and 21000 BF16 shapes of up to 256 tiles of
// 128 x 128 while those had four waves.  With eight, over 6000 FP8 shapes: what they choose is 0.2 % slower on average than the fastest of all kernels, and more than 3 %
// slower than without small tiles on 0.9 % of them (0.3 % with four waves), more than 10 % on 0.1 %.  Taking 0.2 to 0.5 us off the times of the larger tile up to 15 K steps chooses no better.
// Every workgroup raises the output absmax, and atomics on one address follow each other.  R x C x T, 128 x 128 / 64 x 64 / 32 x 32:
//   256 x 1024 x 512 5.4 / 5.1 / 4.1, with absmax (four waves) 5.2 / 5.2 / 6.0;  256 x 512 x 1024 6.6 / 5.9 / 4.4;  1024 x 512 x 256 4.9 / 5.2 / 6.3;
//   128 x 256 x 6688 21.0 / 15.8 / 9.0, 117 x 304 x 14496 40.7 / 28.7 / 15.0, 128 x 1792 x 19456 53.2 / 37.8 / 19.4, 448 x 512 x 3584 13.1 / 10.1 / 6.5,
//   16 x 4096 x 4096 14.2 / 10.3 / 6.6, 862 x 768 x 3008 12.5 / 9.9 / 15.2, 1024 x 1024 x 4096 14.6 / 12.5 / 24.6, 128 x 8192 x 1024 7.1 / 6.4 / 12.3,
//   1024 x 2048 x 2048 10.2 / 14.2 / 28.2
// generic / 64 x 64 / 32 x 32 of short contractions: 1 x 1 x 256 2.4 / 3.5 / 3.2, 624 x 689 x 224 4.1 / 5.7 / -, 3456 x 128 x 160 3.9 / 4.8 / -, 300 x 300 x 64
//   2.8 / 4.6 / 3.5, 100 x 136 x 512 4.3 / 4.9 / 3.5;  added to what is there 88 x 17 x 64 3.2 / 4.3 / 4.0, 206 x 1326 x 128 4.7 / 8.2 / 7.5
// shared_us: what the contraction takes with its left-over tiles shared out (shared_tiles_us), 0 if they are not.  Operands beyond the
// 256 MB memory-side cache slow the small tiles down.  128 x 128 tiles shared out / small tiles: 512 x 512 x 131072 246 / 127 us, x 262144 283 / 288;
//   512 x 1024 x 65536 144 / 120, x 131072 178 / 276;  1024 x 1024 x 32768 93 / 62, x 65536 117 / 145, x 262144 275 / 596;  1024 x 2048 x 8192 62 / 37,
//   x 32768 93 / 119
// LLMQ_GEMM_MINI=32 / 64 / 0 (tests): that side wherever the operands allow it, or never.
inline int takes_mini(int64_t R, int64_t C, int64_t T, bool slabs_a, bool slabs_b, bool accumulate, bool with_amax, bool bf16, int num_cus, double shared_us = 0.0) {
    if (T >= (1ll << 23) || R >= (1ll << 23) || C >= (1ll << 23) || T < 16 || (!(slabs_a && slabs_b) && T % 16 != 0)) return 0;
    const int64_t tiles128 = ((R + 127) / 128) * ((C + 127) / 128);
    if (tiles128 > ((int64_t)1 << 20)) return 0;                          // (32 x 32 tiles then fit a launch)
    if (const char* e = tuning_env("LLMQ_GEMM_MINI")) { const int side = atoi(e); return side == 32 || side == 64 ? side : 0; }
    if (tuning_env("LLMQ_GEMM_TILE") || tuning_env("LLMQ_GEMM_EDGE_TILE") || tuning_env("LLMQ_GEMM_ANY_TILE") || tuning_env("LLMQ_GEMM_DEEP") || tuning_env("LLMQ_GEMM_SPLIT")) return 0;     // (tests of the other kernels)
    if (tiles128 > num_cus) return 0;
    const double slower = shared_us > 0.0 && (R + C) * T > 100000000 ? 1.25 : 1.0;
    double best = (shared_us > 0.0 ? shared_us : other_tiles_us(R, C, T, accumulate, with_amax, bf16, num_cus)) - 0.2;       // (a margin for the models' errors)
    int side = 0;
    for (int s = 64; s >= 32; s -= 32) {
        const double cost = slower * small_tiles_us(s, R, C, T, accumulate, with_amax, num_cus);
        if (cost < best) { best = cost; side = s; }
    }
    return side;
}

// Whether a weight gradient reads the row-major copies T-major (as under LLMQ_NO_TRANSPOSE; same bytes) although the transposed
// ones are there: with a token count that is no multiple of 16 the rows of those start at any address, so their chunks go through
// registers and touch two cache lines each, while the row-major copies' rows are as long as the layer is wide.  Transposed /
// row-major copies, N x K x M, microseconds:
//   M no multiple of 16   7168 x 5120 x 8100 355 / 219, 2880 x 960 x 1777 20.1 / 11.1, 3072 x 3072 x 105 21.2 / 9.9, 512 x 512 x 17 6.1 / 4.7
//     widths no multiples of 16 either: as aligned as the rows of the copies are (1, 2, or 4 and more bytes: in dwords), over 3000 shapes of more than
//     one K step, transposed / row-major time with M odd 1.07 to 1.36;  M a multiple of 2, both widths of 2 1.05, one odd and the other of 16 1.12, both
//     odd 0.98;  M a multiple of 4 or 8, both widths of 4 1.03 to 1.12, one odd 0.88 to 1.00 (739 x 7055 x 8476 86 / 111, 139 x 75 x 2804 17.9 / 24.5)
//     one K step: the generic kernel, 300 x 300 x 127 7.3 / 9.4
//   M a multiple of 16, not of 64 (aligned chunks over two lines)   7168 x 5120 x 8112 273 / 232; operands that an XCD's 4 MB L2 holds lose, 1024 x 512 x
//     2032 8.0 / 9.7; and where the transposed copies' small tiles are taken, they are the faster ones: 1024 x 512 x 8112
//     25.3 / 28.0, 1024 x 512 x 4016 15.1 / 15.1, 512 x 512 x 8112 11.8 / 24.8, 304 x 256 x 14496 17.3 / 54.3, 1536 x 448 x 12560 38.8 / 42.4
//   M a multiple of 64   8128: 3072 x 3072 82.8 / 70.0, 14496 x 304 64 / 63;  640 x 384 x 640 4.5 / 5.9: left as they are
inline bool wgrad_reads_row_major(int64_t M, int64_t N, int64_t K, bool accumulate, int num_cus) {
    if (M % 64 == 0 || M < 16 || N < 16 || K < 16) return false;
    const int64_t lim = 0x7FFFFF00ll - ((int64_t)1 << 24);           // what the T-major tile kernels address
    if ((M + 256) * N >= lim || (M + 256) * K >= lim) return false;
    const bool whole_chunks = N % 16 == 0 && K % 16 == 0;
    if (M % 16 == 0) return whole_chunks && M * (N + K) > ((int64_t)4 << 20) && takes_mini(N, K, M, false, false, accumulate, false, false, num_cus) == 0;
    if (whole_chunks || M <= 128) return whole_chunks;
    if (M % 2 != 0 || (N % 4 == 0 && K % 4 == 0)) return true;
    return M % 4 != 0 && ((N % 2 == 0 && K % 2 == 0) || N % 16 == 0 || K % 16 == 0);
}

}  // namespace llmq

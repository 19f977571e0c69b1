// Host-side brute force over the index arithmetic of the tile kernel's launches, under the sanitizers: the walk
// of the workgroup ids over the tiles, the planner that shares a ragged last round of tiles among the compute
// units, the walk of the quantize kernel's workgroups over the blocks of its tensor, that of the 64 x 128-tile kernels'
// workgroups over their tiles, and the kernels that shapes which were timed in all of them are given.  Every tile, and every K step of every shared tile, must be computed exactly once, and every partial
// result must have a slot of its own inside the scratch the plan asks for.
#include <stdio.h>
#include <stdlib.h>

#include <vector>

#include "../../paper_2512_15306_amd/csrc/gemm_tile.h"
#include "../../paper_2512_15306_amd/csrc/llmq_device.h"

using namespace llmq;

static int g_fail = 0;
#define CHECK(cond, ...)                                  \
    do {                                                  \
        if (!(cond)) {                                    \
            if (g_fail < 20) { printf("FAIL %s:%d %s: ", __FILE__, __LINE__, #cond); printf(__VA_ARGS__); printf("\n"); } \
            ++g_fail;                                     \
        }                                                 \
    } while (0)

static void check_walk(int n) {
    const int grid = ((n + kXcds - 1) / kXcds) * kXcds;
    std::vector<int> seen(n, 0);
    for (int pid = 0; pid < grid; ++pid) {
        const int pos = walk_position(pid, n);
        CHECK(pos >= -1 && pos < n, "n=%d pid=%d pos=%d", n, pid, pos);
        if (pos >= 0) ++seen[pos];
    }
    for (int p = 0; p < n; ++p) CHECK(seen[p] == 1, "n=%d position %d taken %d times", n, p, seen[p]);
    // workgroups of one XCD (ids congruent modulo the XCD count) take neighbouring positions in id order
    for (int pid = kXcds; pid < grid; ++pid) {
        const int a = walk_position(pid - kXcds, n), b = walk_position(pid, n);
        if (a >= 0 && b >= 0) CHECK(b == a + 1, "n=%d pid=%d: %d after %d", n, pid, b, a);
    }
}

static void check_tiles(int tiles_r, int tiles_c, int band) {
    const int nt = tiles_r * tiles_c;
    std::vector<int> seen(nt, 0);
    for (int pos = 0; pos < nt; ++pos) {
        int tr = -1, tc = -1;
        tile_of_position(pos, tiles_r, tiles_c, band, tr, tc);
        CHECK(tr >= 0 && tr < tiles_r && tc >= 0 && tc < tiles_c, "%d x %d band %d pos %d -> (%d, %d)", tiles_r, tiles_c, band, pos, tr, tc);
        if (tr >= 0 && tr < tiles_r && tc >= 0 && tc < tiles_c) ++seen[tr * tiles_c + tc];
    }
    for (int t = 0; t < nt; ++t) CHECK(seen[t] == 1, "%d x %d band %d: tile %d computed %d times", tiles_r, tiles_c, band, t, seen[t]);
}

// The walk of the quantize kernel's workgroups over the blocks of its tensor (band_walk): a bijection, also for the
// grids of very tall tensors, where band x grid_rows comes close to 2^32.
static void check_bands(unsigned gr, unsigned gc, unsigned band) {
    if (band > gc) band = gc;                      // as the launcher does
    const unsigned long long n = (unsigned long long)gr * gc;
    std::vector<unsigned char> seen(n, 0);
    for (unsigned long long id = 0; id < n; ++id) {
        unsigned br = ~0u, bc = ~0u;
        band_walk((unsigned)id, gr, gc, band, br, bc);
        CHECK(br < gr && bc < gc, "grid %u x %u band %u: id %llu -> (%u, %u)", gr, gc, band, id, br, bc);
        if (br < gr && bc < gc) {
            CHECK(seen[(size_t)br * gc + bc] == 0, "grid %u x %u band %u: block (%u, %u) twice", gr, gc, band, br, bc);
            seen[(size_t)br * gc + bc] = 1;
        }
    }
}

// The 64 x 128-tile kernels: every tile once, whatever the launches are cut into; no id but the padding ones without a tile, id 0
// with one (it stores the scale); on ragged pitches each XCD's ids (congruent modulo 8) on one contiguous range of the walk.
static void check_small(int64_t rows, int64_t cols, bool transposed) {
    const SmallGrid g = small_grid(rows, cols, false, transposed);
    CHECK(g.rows == (unsigned)((rows + 63) / 64) && g.cols == (unsigned)((cols + 127) / 128) && g.first == 0, "%lld x %lld", (long long)rows, (long long)cols);
    CHECK(g.blocks % 8 == 0 && g.blocks >= g.rows * g.cols && g.blocks < g.rows * g.cols + 8, "%lld x %lld: %u workgroups", (long long)rows, (long long)cols, g.blocks);
    std::vector<int> seen((size_t)g.rows * g.cols, 0), in_launches(g.blocks, 0);
    small_launches(g, [&](const SmallGrid& part, unsigned n) {
        for (unsigned b = 0; b < n; ++b) {
            const unsigned id = part.first + b;
            CHECK(id < g.blocks, "id %u of %u", id, g.blocks);
            if (id < g.blocks) ++in_launches[id];
        }
    });
    unsigned padding = 0;
    for (unsigned id = 0; id < g.blocks; ++id) {
        CHECK(in_launches[id] == 1, "%lld x %lld: id %u launched %d times", (long long)rows, (long long)cols, id, in_launches[id]);
        unsigned br = ~0u, bc = ~0u;
        if (!small_tile(g, id, br, bc)) { ++padding; CHECK(id != 0, "id 0 without a tile"); continue; }
        CHECK(br < g.rows && bc < g.cols, "%lld x %lld id %u -> (%u, %u)", (long long)rows, (long long)cols, id, br, bc);
        if (br < g.rows && bc < g.cols) ++seen[(size_t)br * g.cols + bc];
        unsigned br2, bc2;
        if (g.xcd_ranges && id + 8 < g.blocks && small_tile(g, id + 8, br2, bc2))          // the next of this XCD: a neighbour in the band or its next row
            CHECK((br2 == br && bc2 == bc + 1) || br2 == br + 1 || br2 == 0, "%lld x %lld: ids %u, %u -> (%u, %u), (%u, %u)", (long long)rows, (long long)cols, id, id + 8, br, bc, br2, bc2);
    }
    CHECK(padding == g.blocks - g.rows * g.cols, "%lld x %lld: %u ids without a tile", (long long)rows, (long long)cols, padding);
    for (size_t t = 0; t < seen.size(); ++t) CHECK(seen[t] == 1, "%lld x %lld: tile %zu taken %d times", (long long)rows, (long long)cols, t, seen[t]);
}

// Replays what the three launches of a contraction do with the plan, as the kernel's prologue does.
static void check_plan(int nt, int nk, int slots, size_t scratch_bytes, const char* mode) {
    const SplitChoice c = choose_split(nt, nk, slots, 4, 4, scratch_bytes);
    const size_t tile_bytes = 4u * 256 * 256;
    CHECK(c.n_whole >= 0 && c.n_whole <= nt, "nt=%d nk=%d %s: n_whole %d", nt, nk, mode, c.n_whole);
    if (c.n_groups == 0) {
        CHECK(c.n_whole == nt, "nt=%d nk=%d %s: nothing shared but n_whole %d", nt, nk, mode, c.n_whole);
        return;
    }
    CHECK(c.n_whole % slots == 0, "nt=%d nk=%d %s: n_whole %d is not whole rounds", nt, nk, mode, c.n_whole);
    CHECK(c.n_whole + c.shared_tiles == nt, "nt=%d nk=%d %s: %d + %d tiles", nt, nk, mode, c.n_whole, c.shared_tiles);
    CHECK(c.n_groups <= kMaxSplitGroups, "groups %d", c.n_groups);
    CHECK(c.slots * tile_bytes <= scratch_bytes, "nt=%d nk=%d %s: %zu slots do not fit %zu bytes", nt, nk, mode, c.slots, scratch_bytes);
    std::vector<int> slot_used(c.slots, 0);
    // steps[t][k]: how often K step k of shared tile t is computed
    std::vector<std::vector<int>> steps(c.shared_tiles, std::vector<int>(nk, 0));
    int tile_at = 0, wg_at = 0;
    bool any_cut = false;
    for (int g = 0; g < c.n_groups; ++g) {
        const SplitGroup& grp = c.group[g];
        CHECK(grp.tile_begin == tile_at && grp.wg_begin == wg_at, "nt=%d nk=%d %s group %d starts at tile %d wg %d, expected %d %d", nt, nk, mode, g, grp.tile_begin, grp.wg_begin, tile_at, wg_at);
        CHECK(grp.tiles >= 1 && grp.pieces >= 1 && grp.steps >= 1, "group %d empty", g);
        CHECK(grp.wgs % kXcds == 0 && grp.wgs >= grp.tiles * grp.pieces, "group %d: %d workgroups for %d x %d", g, grp.wgs, grp.tiles, grp.pieces);
        CHECK(grp.pieces == 1 || grp.tiles * grp.pieces <= slots, "nt=%d nk=%d %s group %d: %d pieces at once on %d slots", nt, nk, mode, g, grp.tiles * grp.pieces, slots);
        CHECK((grp.pieces - 1) * grp.steps < nk && grp.pieces * grp.steps >= nk, "nt=%d nk=%d %s group %d: %d pieces of %d steps", nt, nk, mode, g, grp.pieces, grp.steps);
        any_cut = any_cut || grp.pieces > 1;
        // the pieces launch
        for (int q = grp.wg_begin; q < grp.wg_begin + grp.wgs; ++q) {
            const int w = walk_position(q - grp.wg_begin, grp.tiles * grp.pieces);
            if (w < 0) continue;
            const int piece = w / grp.tiles, j = w - piece * grp.tiles;
            const int kb = piece * grp.steps;
            int n = nk - kb < grp.steps ? nk - kb : grp.steps;
#ifdef LLMQ_PLANT_SHORT_PIECES      // a replay that drops the last K step of every last piece: the checks must notice
            if (grp.pieces > 1 && piece == grp.pieces - 1) --n;
#endif
            CHECK(n >= 0, "nt=%d nk=%d %s group %d: empty piece %d", nt, nk, mode, g, piece);
#ifndef LLMQ_PLANT_SHORT_PIECES
            CHECK(n > 0, "nt=%d nk=%d %s group %d: empty piece %d", nt, nk, mode, g, piece);
#endif
            const int slot = grp.wg_begin + j * grp.pieces + piece;
            CHECK(slot >= 0 && (size_t)slot < c.slots, "slot %d of %zu", slot, c.slots);
            if (slot >= 0 && (size_t)slot < c.slots) ++slot_used[slot];
            for (int k = kb; k < kb + n && k < nk; ++k) ++steps[grp.tile_begin + j][k];
        }
        // the fix-up launch reads slots [first, first + pieces) of tile j in this order
        for (int j = 0; j < grp.tiles; ++j) {
            const int first = grp.wg_begin + j * grp.pieces;
            for (int p = 0; p < grp.pieces; ++p) CHECK(slot_used[first + p] == 1, "nt=%d nk=%d %s group %d tile %d piece %d: slot written %d times", nt, nk, mode, g, j, p, slot_used[first + p]);
        }
        tile_at += grp.tiles;
        wg_at += grp.wgs;
    }
    CHECK(tile_at == c.shared_tiles && wg_at == c.share_wgs, "nt=%d nk=%d %s: groups hold %d tiles %d workgroups, plan says %d %d", nt, nk, mode, tile_at, wg_at, c.shared_tiles, c.share_wgs);
    CHECK(any_cut, "nt=%d nk=%d %s: a plan that cuts nothing", nt, nk, mode);
    for (int t = 0; t < c.shared_tiles; ++t)
        for (int k = 0; k < nk; ++k) CHECK(steps[t][k] == 1, "nt=%d nk=%d %s: K step %d of shared tile %d computed %d times", nt, nk, mode, k, t, steps[t][k]);
}

// Which tile side, or another kernel (0), contractions of few outputs take: the fastest one where all were timed.
struct SmallCase { int64_t R, C, T; bool accumulate, with_amax, bf16; int side; };      // T in bytes
static void check_small_tiles() {
    const SmallCase cases[] = {
        // BF16, eight elements: a lane per output is done before a tile has been loaded
        {1, 1, 16, false, false, true, 0}, {48, 2720, 16, false, false, true, 0}, {300, 300, 16, false, false, true, 0}, {128, 640, 16, true, false, true, 0},
        {40, 40, 48, false, false, true, 32}, {100, 136, 64, false, false, true, 32}, {256, 1024, 1024, false, false, true, 32},
        {448, 512, 3584, false, false, true, 32}, {1024, 1024, 4096, false, false, true, 64},
        // FP8: short contractions whose generic waves or 128 x 128 tiles are done first, added to the output or not
        {1, 1, 256, false, false, false, 0}, {300, 300, 64, false, false, false, 0}, {624, 689, 224, false, false, false, 0}, {3456, 128, 160, false, false, false, 0},
        {1344, 518, 192, false, false, false, 0}, {88, 17, 64, true, false, false, 0}, {206, 1326, 128, true, false, false, 0}, {977, 264, 128, true, false, false, 0},
        {1600, 325, 96, true, false, false, 0}, {128, 19, 32, true, true, false, 0}, {84, 128, 128, false, true, false, 0}, {896, 384, 384, false, false, false, 64},
        {100, 136, 512, false, false, false, 32}, {256, 1024, 512, false, false, false, 32}, {128, 256, 6688, true, false, false, 32},
        {1024, 1024, 4096, false, false, false, 64}, {128, 8192, 1024, false, false, false, 64}, {1024, 2048, 2048, false, false, false, 0},
    };
    for (const SmallCase& c : cases) {
        const int side = takes_mini(c.R, c.C, c.T, false, false, c.accumulate, c.with_amax, c.bf16, 256);
        CHECK(side == c.side, "%lld x %lld x %lld acc %d amax %d bf16 %d: side %d, measured best %d", (long long)c.R, (long long)c.C, (long long)c.T, c.accumulate, c.with_amax, c.bf16, side, c.side);
    }
    // long contractions with scratch, which 256 x 256 tiles share out: the faster of that and the small tiles
    const SmallCase shared[] = {{512, 512, 131072, false, false, false, 32}, {512, 1024, 65536, false, false, false, 32}, {512, 1024, 131072, false, false, false, 0},
                                {1024, 1024, 32768, false, false, false, 64}, {1024, 1024, 65536, false, false, false, 0}, {1024, 1024, 262144, false, false, false, 0},
                                {256, 2048, 131072, false, false, false, 0}, {1024, 2048, 8192, false, false, false, 64}, {1024, 2048, 32768, false, false, false, 0},
                                {256, 256, 262144, false, false, false, 32}};
    for (const SmallCase& c : shared) {
        const double us = shared_tiles_us(choose_split((int)((c.R / 256) * (c.C / 256)), (int)(c.T / BK), 256, 4, 4, (size_t)1 << 30));
        const int side = takes_mini(c.R, c.C, c.T, false, false, false, false, false, 256, us);
        CHECK(us > 0.0 && side == c.side, "%lld x %lld x %lld shared out in %.0f us: side %d, measured best %d", (long long)c.R, (long long)c.C, (long long)c.T, us, side, c.side);
    }
}

// Which copies a weight gradient [N, K] of M tokens reads: those it is faster on, by measurement.
static void check_wgrad_copies() {
    struct Case { int64_t N, K, M; bool accumulate, row_major; };
    const Case cases[] = {
        // whole chunks either way: the transposed copies where the small tiles take them, the row-major ones of larger layers
        {1024, 512, 8112, false, false}, {1024, 512, 4016, false, false}, {512, 512, 8112, false, false}, {304, 256, 14496, false, false}, {1536, 448, 12560, true, false},
        {2880, 960, 1776, false, true}, {512, 2432, 2336, false, true}, {832, 3776, 16272, true, true}, {7168, 5120, 8112, false, true}, {1024, 512, 2032, false, false},
        // rows of the transposed copies at any address
        {7168, 5120, 8100, false, true}, {2880, 960, 1777, false, true}, {512, 512, 17, false, true}, {1001, 1003, 4001, false, true}, {300, 300, 127, false, false},
        // ... and widths too: the better aligned of the two
        {739, 7055, 8476, false, false}, {139, 75, 2804, false, false}, {69, 256, 3812, false, false}, {141, 255, 2062, false, false}, {1733, 202, 6728, false, false},
        {164, 36, 4220, false, true}, {1544, 8, 9272, false, false}, {1544, 24, 9272, false, true}, {6058, 540, 1374, false, true}, {117, 1104, 6558, false, true}, {502, 4866, 147, false, true},
        {3072, 3072, 8128, false, false}, {640, 384, 640, false, false}, {15, 512, 8100, false, false},
    };
    for (const Case& c : cases) CHECK(wgrad_reads_row_major(c.M, c.N, c.K, c.accumulate, 256) == c.row_major, "weight gradient %lld x %lld of %lld tokens", (long long)c.N, (long long)c.K, (long long)c.M);
}

// Tiles of ragged contractions: 192 x 128 against 128 x 128 tiles that are all resident, the faster one by measurement.
static void check_edge_tiles() {
    struct Case { int64_t R, C, T; bool tb, accumulate, with_amax, bf16; int ni, nj; };
    const Case cases[] = {
        {5477, 945, 128, false, true, false, false, 2, 2}, {2448, 1566, 96, false, true, false, false, 2, 2}, {896, 6208, 16, false, true, false, false, 2, 2},
        {7232, 704, 112, true, true, false, false, 2, 2}, {2176, 2624, 16, true, true, false, false, 2, 2}, {6936, 555, 64, false, false, false, true, 2, 2},
        {768, 5509, 32, false, true, false, true, 2, 2}, {1466, 3335, 256, false, false, false, true, 2, 2}, {2432, 2048, 720, false, false, false, false, 3, 2},
        {708, 7536, 640, false, false, false, false, 3, 2}, {576, 9600, 736, false, false, false, false, 3, 2}, {4480, 2432, 3760, false, false, false, false, 3, 4},
        {7296, 1060, 3712, false, false, false, false, 3, 4}, {7105, 4754, 64, false, true, false, false, 2, 2},
    };
    for (const Case& c : cases) {
        const EdgeChoice e = choose_edge_tile(c.R, c.C, c.T, 256, false, c.tb, false, false, c.accumulate, c.with_amax, c.bf16);
        CHECK(e.ni == c.ni && e.nj == c.nj && e.edge == kEdge, "%lld x %lld x %lld: %d x %d, measured best %d x %d", (long long)c.R, (long long)c.C, (long long)c.T, e.ni, e.nj, c.ni, c.nj);
    }
}

// Large tiles and guarded ones in place of the tile chosen before: the faster one by measurement, and none where the guarded form does not exist.
static void check_better_tiles() {
    struct Case { int64_t R, C, T; bool ta, tb, accumulate; TilePlan base, best; };
    const Case cases[] = {
        {8192, 5120, 13824, false, false, false, {4, 4, kNoEdge}, {4, 5, kNoEdge}}, {4096, 5120, 3072, false, false, false, {4, 4, kNoEdge}, {4, 5, kNoEdge}},
        {6144, 6656, 6144, false, false, true, {4, 4, kNoEdge}, {4, 5, kEdge}},     {12160, 3328, 960, false, false, true, {2, 2, kEdge}, {5, 4, kEdge}},
        {4480, 2176, 8320, false, false, false, {2, 2, kNoEdge}, {3, 4, kEdge}},    {1792, 7552, 4096, false, false, true, {2, 2, kNoEdge}, {4, 4, kEdge}},
        {3584, 5632, 7680, false, true, false, {2, 2, kNoEdge}, {4, 5, kEdge}},     {4480, 13184, 3072, true, true, false, {2, 2, kNoEdge}, {5, 4, kEdge}},
        {6400, 2432, 5120, true, true, false, {2, 2, kNoEdge}, {4, 4, kEdge}},
        // the tile they have
        {4080, 2816, 544, false, false, false, {3, 4, kEdge}, {3, 4, kEdge}},       {5376, 5376, 256, false, false, true, {4, 4, kNoEdge}, {4, 4, kNoEdge}},
        {1600, 16128, 608, false, false, false, {4, 4, kEdge}, {4, 4, kEdge}},      {4864, 1536, 5632, false, false, false, {2, 2, kNoEdge}, {2, 2, kNoEdge}},
        {12288, 2304, 11776, false, false, true, {4, 4, kNoEdge}, {4, 4, kNoEdge}}, {2048, 2048, 2048, false, false, false, {2, 2, kNoEdge}, {2, 2, kNoEdge}},
        // added to the output, which costs the large tiles most; and 128 x 192 tiles, which are two to a CU
        {3232, 43520, 480, false, true, true, {4, 4, kEdge}, {4, 4, kEdge}},        {3072, 46080, 336, false, false, true, {4, 4, kEdge}, {4, 4, kEdge}},
        {3232, 43624, 384, false, false, true, {4, 4, kEdge}, {4, 4, kEdge}},
        {12288, 2496, 256, false, false, false, {2, 3, kNoEdge}, {2, 3, kNoEdge}},  {12928, 576, 384, false, false, true, {2, 3, kNoEdge}, {2, 3, kNoEdge}},
        {896, 25920, 384, false, true, false, {2, 3, kNoEdge}, {2, 3, kNoEdge}},    {22784, 576, 256, false, false, true, {2, 3, kNoEdge}, {2, 3, kNoEdge}},
        {22144, 4800, 640, false, false, false, {2, 3, kNoEdge}, {2, 3, kNoEdge}},
        // widths that are no multiples of 8: the tile they have where the contraction is short, large ones where they save a round or the contraction is long
        {1536, 38369, 256, false, false, false, {4, 4, kEdge}, {5, 4, kEdge}},      {768, 45462, 384, false, false, false, {2, 2, kEdge}, {2, 2, kEdge}},
        {8160, 4982, 448, false, false, false, {2, 2, kEdge}, {2, 2, kEdge}},       {9344, 3932, 512, false, false, false, {2, 2, kEdge}, {2, 2, kEdge}},
        {1376, 26375, 768, false, false, false, {2, 2, kEdge}, {2, 2, kEdge}},      {2304, 7778, 1152, false, false, false, {3, 2, kEdge}, {3, 2, kEdge}},
        {736, 27066, 384, false, false, true, {2, 2, kEdge}, {2, 2, kEdge}},        {1792, 10561, 304, false, false, true, {2, 2, kEdge}, {2, 2, kEdge}},
        {8960, 5812, 1024, false, false, false, {4, 4, kEdge}, {5, 4, kEdge}},      {7424, 18060, 256, false, false, false, {4, 4, kEdge}, {5, 4, kEdge}},
        {5888, 3070, 5872, false, false, true, {3, 2, kEdge}, {5, 4, kEdge}},       {3917, 13994, 4480, false, false, false, {4, 4, kEdge}, {5, 4, kEdge}},
        // A T-major alone, rows that are not whole chunks, one K step, rows beyond 32-bit offsets, the generic kernel
        {4096, 5120, 3072, true, false, false, {4, 4, kNoEdge}, {4, 4, kNoEdge}},   {4096, 5121, 3072, false, true, false, {4, 4, kEdgeUnaligned}, {4, 4, kEdgeUnaligned}},
        {4096, 5120, 3073, false, false, false, {4, 4, kEdgeUnaligned}, {4, 4, kEdgeUnaligned}}, {4096, 5120, 128, false, false, false, {4, 4, kNoEdge}, {4, 4, kNoEdge}},
        {4096, 5120, 1 << 22, false, false, false, {4, 4, kNoEdge}, {4, 4, kNoEdge}}, {300, 300, 64, false, false, false, {0, 0, kNoEdge}, {0, 0, kNoEdge}},
    };
    for (const Case& c : cases) {
        const TilePlan p = better_tile(c.R, c.C, c.T, 256, c.ta, c.tb, false, false, c.accumulate, c.base, 1.0);
        CHECK(p.ni == c.best.ni && p.nj == c.best.nj && p.edge == c.best.edge, "%lld x %lld x %lld: %d x %d form %d, measured best %d x %d form %d", (long long)c.R, (long long)c.C,
              (long long)c.T, p.ni, p.nj, p.edge, c.best.ni, c.best.nj, c.best.edge);
    }
}

// Whose first slabs a workgroup requests: those of the one that takes its place, in long launches of tiles that have a CU to themselves.
static void check_successors() {
    for (int ni = 2; ni <= 5; ++ni)
        for (int nj = 2; nj <= 5; ++nj) {
            const int slots = resident_slots(256, ni, nj);
            const int lds = 2 * (64 * ni + 64 * nj) * BK;
            CHECK(alone_on_cu(ni, nj) == (2 * lds > 160 * 1024), "%d x %d", ni, nj);
            CHECK(successor_stride(ni, nj, 6 * slots, slots) == (2 * lds > 160 * 1024 ? 256 : 0) && successor_stride(ni, nj, 6 * slots - 1, slots) == 0, "%d x %d", ni, nj);
        }
}

// A problem whose last round is shared out stays so, or is computed whole on larger tiles, whether its output is added to or not.
static void check_shared_choice() {
    int kept = 0, replaced = 0;
    for (int64_t r = 4; r <= 64; r += 3)
        for (int64_t c = 4; c <= 110; c += 5)
            for (int64_t t = 64; t <= 1024; t *= 2) {
                const SplitChoice sc = choose_split((int)(r * c), (int)t, 256, 4, 4, ~(size_t)0);
                if (sc.n_groups == 0) continue;
                const TilePlan base{4, 4, kNoEdge};
                const double scale = sc.cost_us / sc.whole_cost_us;
                const TilePlan p = better_tile(256 * r, 256 * c, BK * t, 256, false, false, false, false, false, base, scale, true);
                const TilePlan q = better_tile(256 * r, 256 * c, BK * t, 256, false, false, false, false, true, base, scale, true);
                CHECK(p.ni == q.ni && p.nj == q.nj, "%lld x %lld x %lld: %d x %d, added to the output %d x %d", (long long)(256 * r), (long long)(256 * c), (long long)(BK * t), p.ni, p.nj, q.ni, q.nj);
                CHECK(p.ni * p.nj == 16 || q.edge == kEdge, "large tiles add to the output in their guarded form");
                ++(p.ni * p.nj == 16 ? kept : replaced);
            }
    CHECK(kept > 100 && replaced > 100, "%d shapes shared out, %d whole", kept, replaced);
}

// How the lanes of the 64 x 128 tile lie, and where codes leave it for the 128 x 128 tile: the faster one by measurement.
static void check_code_tiles() {
    struct Case { int64_t rows, cols; bool quantizes, stacked; };
    const Case cases[] = {{16221, 4296, true, true}, {9579, 11200, true, true}, {12446, 5904, true, true}, {11001, 3912, true, true}, {12001, 5000, true, true},
                          {9001, 4008, true, false}, {8101, 4416, true, false}, {8100, 7168, true, false}, {4133, 5120, true, false}, {1777, 2730, true, false},
                          {16001, 8001, true, false}, {12545, 8008, false, true}, {12001, 5000, false, false}, {12545, 8001, false, false}, {1777, 960, false, false}};
    for (const Case& c : cases) CHECK(small_grid(c.rows, c.cols, c.quantizes, true).stacked == c.stacked, "lanes for %lld x %lld (quantize %d)", (long long)c.rows, (long long)c.cols, c.quantizes);
    struct Alone { int64_t rows, cols; bool ranges; };          // without the transposed copy
    const Alone alone[] = {{13543, 9984, false}, {12005, 7488, false}, {10134, 3840, false}, {357, 16064, true}, {6762, 2752, true}, {9254, 7448, true}, {10043, 14456, true}, {12001, 5001, true}};
    for (const Alone& c : alone) {
        const SmallGrid g = small_grid(c.rows, c.cols, false, false);
        CHECK(g.xcd_ranges == c.ranges && !g.stacked, "codes alone of %lld x %lld", (long long)c.rows, (long long)c.cols);
    }
    struct Tiles { int64_t rows, cols; LargeTiles range; bool large; };
    const Tiles tiles[] = {{1024, 4096, kQuantizeTiles, true}, {1024, 4100, kQuantizeTiles, false}, {1024, 2048, kQuantizeTiles, false}, {1920, 8192, kQuantizeTiles, true},
                           {1024, 4096, kNormTiles, false}, {2048, 2560, kNormTiles, false}, {2048, 4096, kNormTiles, false}, {2432, 5120, kNormTiles, true}, {2816, 4480, kNormTiles, false},
                           {1920, 8192, kNormTiles, false}, {1152, 14336, kNormTiles, false}, {1664, 10752, kNormTiles, true}, {3456, 5376, kNormTiles, true}, {16384, 5120, kNormTiles, true},
                           {1024, 4096, kNormOutputTiles, false}, {2048, 2560, kNormOutputTiles, true}, {2048, 4096, kNormOutputTiles, true}, {1920, 8192, kNormOutputTiles, true},
                           {1024, 4096, kSwigluTiles, true}, {2048, 2560, kSwigluTiles, false}, {2048, 4096, kSwigluTiles, false}, {2048, 5120, kSwigluTiles, false}, {2304, 5120, kSwigluTiles, true},
                           {1024, 2048, kSwigluTiles, false}, {1024, 4096, kSwigluOutputTiles, true}, {2048, 2560, kSwigluOutputTiles, false}, {2048, 3072, kSwigluOutputTiles, false},
                           {2816, 2560, kSwigluOutputTiles, true}, {2048, 5120, kSwigluOutputTiles, true}};
    for (const Tiles& c : tiles)
        CHECK(takes_large_tile(c.rows, c.cols, c.range) == c.large, "128 x 128 tiles for %lld x %lld, from %lld", (long long)c.rows, (long long)c.cols, (long long)c.range.least);
}

// Widths that are no multiples of 8: every LDS read of the guarded epilogue, as it computes them, lies in the wave's stage of 32 rows however far the edge of
// the output is, and every column of the wave's tile that exists is read by one lane.
template <int SLOTS>
static void check_staged_columns() {
    const bool rest = kWave % SLOTS != 0;
    const int width = 8 * SLOTS, pitch = 32 * SLOTS + (rest ? 16 : 0);
    for (int cols_left = 1; cols_left < (1 << 22); cols_left += cols_left < 3 * width ? 1 : cols_left / 7) {
        std::vector<int> seen(width, 0);
        for (int cc = 0; cc < width && cc < cols_left; cc += kWave)
            for (int lane = 0; lane < kWave; ++lane) {
                const int c = width % kWave == 0 || cc + lane < width ? cc + lane : cols_left, from = staged_column<SLOTS>(c);
                CHECK(c >= 0 && (c < width || c >= cols_left), "%d pieces, %d columns left: lane %d of trip %d at column %d", SLOTS, cols_left, lane, cc, c);
                if (c < cols_left && c < width) { ++seen[c]; CHECK(from == c, "column %d read at %d", c, from); }
                for (int r = 0; r < 32; ++r) {
                    const int at = ((from >> 2) & 1) * (16 * SLOTS) + (from & 3) * 4 + r * pitch + ((rest ? from >> 3 : ((from >> 3) + r) % SLOTS) << 4);
                    CHECK(at >= 0 && at + 4 <= 32 * pitch, "%d pieces, %d columns left: lane %d of trip %d reads byte %d of %d", SLOTS, cols_left, lane, cc, at, 32 * pitch);
                }
            }
        for (int c = 0; c < width && c < cols_left; ++c) CHECK(seen[c] == 1, "%d pieces, %d columns left: column %d moved by %d lanes", SLOTS, cols_left, c, seen[c]);
    }
}

int main() {
    check_staged_columns<4>();            // 128 x 128 tiles of eight waves
    check_staged_columns<8>();
    check_staged_columns<16>();
    check_staged_columns<20>();           // 256 x 320
    check_small_tiles();
    check_code_tiles();
    check_wgrad_copies();
    check_edge_tiles();
    check_better_tiles();
    check_shared_choice();
    check_successors();
    for (int n = 1; n <= 1100; n += (n < 300 ? 1 : 37)) check_walk(n);
    check_walk(13824);
    const int bands[] = {1, 2, 3, 4, 8, 64};
    for (int r = 1; r <= 40; r += (r < 10 ? 1 : 7))
        for (int c = 1; c <= 220; c += (c < 10 ? 1 : 23))
            for (int b : bands) check_tiles(r, c, b);
    check_tiles(64, 216, 4);
    const unsigned band_sizes[] = {1, 2, 3, 7, 16, 1u << 20};
    for (unsigned gr : {1u, 2u, 5u, 64u, 130u})
        for (unsigned gc : {1u, 2u, 3u, 14u, 20u, 33u})
            for (unsigned b : band_sizes) check_bands(gr, gc, b);
    for (unsigned b : band_sizes) {
        check_bands(4096, 20, b);                  // 524288 rows: 2^20 x 4096 would wrap to 0 without the clamp
        check_bands(3 * 4096 + 1, 7, b);
        check_bands(1u << 20, 2, b);               // 2^27 rows
    }
    for (const char* most : {(const char*)nullptr, "8", "64"}) {
        if (most) setenv("LLMQ_MAX_WORKGROUPS", most, 1);
        else unsetenv("LLMQ_MAX_WORKGROUPS");
        for (int64_t r : {1, 64, 65, 130, 640, 1025, 5000})
            for (int64_t c : {1, 24, 128, 129, 192, 1000, 1024, 1152, 1300, 4097, 9000}) { check_small(r, c, true); check_small(r, c, false); }
    }
    unsetenv("LLMQ_MAX_WORKGROUPS");
    const char* modes[] = {nullptr, "1", "a2", "a3", "a5", "a16", "0"};
    const int nks[] = {1, 2, 7, 8, 15, 16, 28, 40, 63, 64, 65, 108, 128, 216, 432};
    const int slot_counts[] = {256, 64, 8};
    for (const char* mode : modes) {
        if (mode) setenv("LLMQ_GEMM_SPLIT", mode, 1);
        else unsetenv("LLMQ_GEMM_SPLIT");
        for (int slots : slot_counts)
            for (int nk : nks)
                for (int nt = 1; nt <= 3 * slots + 5; nt += (slots > 64 && nt > 20 ? 3 : 1)) {
                    check_plan(nt, nk, slots, (size_t)1 << 40, mode ? mode : "default");
                    check_plan(nt, nk, slots, (size_t)64 << 20, mode ? mode : "default");      // 256 binary32 tiles
                    check_plan(nt, nk, slots, 0, mode ? mode : "default");
                }
    }
    unsetenv("LLMQ_GEMM_SPLIT");
    // what the default rule shares: long contractions whose left-over tiles fit one group
    CHECK(choose_split(560, 128, 256, 4, 4, (size_t)1 << 40).n_groups == 1, "560 tiles x 128 steps");
    CHECK(choose_split(560, 128, 256, 4, 4, 0).n_groups == 0, "no scratch, no sharing");
    CHECK(choose_split(448, 296, 256, 4, 4, (size_t)1 << 40).n_groups == 0, "192 left-over tiles need two groups");
    CHECK(choose_split(560, 40, 256, 4, 4, (size_t)1 << 40).n_groups == 0, "short contraction");
    CHECK(choose_split(512, 128, 256, 4, 4, (size_t)1 << 40).n_groups == 0, "whole rounds");
    if (g_fail) { printf("%d checks failed\n", g_fail); return 1; }
    printf("planner driver ok\n");
    return 0;
}

// Tile forms of the GEMM launches with few token rows, and the rule that picks one.  Plain C++17, no HIP
// types, so that a host program can walk the rule (tests/gemm_forms_check.cpp).
//
// X(TM, TN, WM, WN, KSUB, NSTG): TM token rows x TN staged weight rows per workgroup, WM x WN wavefronts
// that multiply, stages of 64 KSUB K-elements, NSTG of them in the LDS ring (mom_gemm_short.hip.inc).
// The smallest tiles take the longest stages (one barrier per stage) and every form a ring that holds
// more than the 32 KiB a CU's vector cache has in flight at most (measured: 256 lines of 128 bytes).
#ifndef MOM_GEMM_FORMS_H
#define MOM_GEMM_FORMS_H

#include <stdint.h>

#define MOM_SHORT_FORMS_DOWN(X)                                                                          \
    X(16, 16, 1, 1, 2, 8) X(32, 16, 2, 1, 4, 6) X(32, 32, 2, 2, 2, 5) X(48, 32, 1, 2, 2, 8)              \
    X(64, 32, 2, 2, 2, 6) X(96, 32, 2, 2, 2, 5) X(128, 32, 4, 1, 1, 8) X(32, 64, 2, 2, 1, 6)             \
    X(64, 64, 2, 2, 1, 5) X(80, 64, 1, 4, 2, 4) X(96, 64, 2, 2, 1, 8) X(128, 64, 2, 2, 1, 6)             \
    X(160, 64, 2, 2, 1, 5) X(192, 64, 2, 2, 1, 5) X(256, 64, 2, 2, 1, 4) X(96, 128, 2, 2, 1, 5)          \
    X(128, 128, 2, 2, 1, 5) X(160, 128, 2, 2, 1, 4) X(192, 128, 2, 2, 1, 4) X(224, 128, 2, 2, 1, 3)
#define MOM_SHORT_FORMS_GATEUP(X)                                                                        \
    X(16, 32, 1, 1, 4, 6) X(32, 32, 2, 1, 2, 8) X(16, 64, 1, 2, 2, 8) X(32, 64, 2, 2, 2, 6)              \
    X(64, 64, 2, 2, 1, 3) X(128, 64, 2, 2, 1, 3) X(64, 128, 2, 2, 1, 6) X(96, 128, 2, 2, 1, 5)           \
    X(128, 128, 2, 2, 1, 5) X(160, 128, 2, 2, 1, 4) X(192, 128, 2, 2, 1, 4) X(224, 128, 2, 2, 1, 3)      \
    X(64, 192, 2, 2, 1, 5) X(96, 192, 2, 2, 1, 4) X(128, 192, 2, 2, 1, 4)

namespace momk {

struct ShortShape { int tm, tn, per_cu; };       // per_cu: workgroups that a CU's 160 KiB of LDS hold
#define MOM_SHAPE(TM, TN, WM, WN, KSUB, NSTG) \
    {TM, TN, 163840 / (NSTG * KSUB * (TM + TN) * 128) > 4 ? 4 : 163840 / (NSTG * KSUB * (TM + TN) * 128)},
constexpr ShortShape kShortDown[] = {MOM_SHORT_FORMS_DOWN(MOM_SHAPE)};
constexpr ShortShape kShortGateUp[] = {MOM_SHORT_FORMS_GATEUP(MOM_SHAPE)};
#undef MOM_SHAPE
constexpr int kShortDownForms = sizeof(kShortDown) / sizeof(kShortDown[0]);
constexpr int kShortGateUpForms = sizeof(kShortGateUp) / sizeof(kShortGateUp[0]);

inline int short_forms(bool gateup) { return gateup ? kShortGateUpForms : kShortDownForms; }
inline ShortShape short_shape(bool gateup, int form) { return gateup ? kShortGateUp[form] : kShortDown[form]; }

// Index of the form with these tiles, or -1.
inline int find_short_form(bool gateup, int tm, int tn) {
    for (int i = 0; i < short_forms(gateup); ++i)
        if (short_shape(gateup, i).tm == tm && short_shape(gateup, i).tn == tn) return i;
    return -1;
}

// Costs are in operand rows x K-elements that one CU moves into its LDS: with few token rows that is what a
// launch takes time for.  A CU's vector cache has 256 lines in flight at most, and at the latency of
// weights that come from HBM that is 55 GB/s, whatever the ring holds and however little is multiplied
// (measured over all forms on 1 ... 2048 rows at K = 14336 and 18944: 0.5 us per operand row at K = 14336,
// i.e. 3.5e-5 us per unit, with a tenth of the spread that the flops per CU have).
// Once per tile: launch, ring prologue, epilogue, 4 us and a little per output element (silu for gate/up);
// the workgroups that share a CU overlap these where the contraction is short.  A 256-row tile 256 weight rows wide, which the matrix
// cores bound, takes as long as 550 operand rows and 9.6 us once.
constexpr double kTileFixed = 115e3, kTileFixedPerGateUp = 5, kTileFixedPerDown = 2;
constexpr double kFullTileRows = 550, kFullTileFixed = 275e3;
// From this contraction length on, what a launch waits for is its operands, not the start and end of tiles.
constexpr int64_t kLongK = 3072;
constexpr int64_t kMaxTiles = 0x1fffffff;            // tile numbers are 32-bit in the kernels

// The tiles of a launch, as it is priced AND as it is launched: tiles_m token tiles in groups of per_group (their
// weights are fetched by one XCD at a time) over group_rows token rows each, tiles_n column tiles.
// (32-bit arithmetic: every launch walks all forms on the host, and M + 1024 < 2^32.)
constexpr int kTokenGroup = 4;
struct TileGrid { uint32_t tiles_m, per_group, group_rows, tiles_n; uint64_t tiles; };
inline TileGrid column_tiles(TileGrid g, int64_t N, uint32_t cols) {
    g.tiles_n = ((uint32_t)N + cols - 1) / cols;
    g.tiles = (uint64_t)g.tiles_m * g.tiles_n;
    return g;
}
// mom_gemm.hip.inc: whole tiles one after the other, only the last one of all is shorter.
inline TileGrid whole_tiles(int64_t rows, int64_t N, uint32_t tm, uint32_t cols) {
    return column_tiles({((uint32_t)rows + tm - 1) / tm, kTokenGroup, kTokenGroup * tm, 0, 0}, N, cols);
}
// mom_gemm_short.hip.inc: the rows spread evenly over the groups, the last tile of each group is shorter.
inline TileGrid spread_tiles(int64_t rows, int64_t N, uint32_t tm, uint32_t cols) {
    const uint32_t M = (uint32_t)rows, most = kTokenGroup * tm;
    uint32_t groups = 1;
    TileGrid g = {0, (M + tm - 1) / tm, M, 0, 0};
    if (M > most) {
        groups = (M + most - 1) / most;
        g.group_rows = (M + groups - 1) / groups;
        groups = (M + g.group_rows - 1) / g.group_rows;
        g.per_group = (g.group_rows + tm - 1) / tm;
    }
    g.tiles_m = (groups - 1) * g.per_group + (M - (groups - 1) * g.group_rows + tm - 1) / tm;
    return column_tiles(g, N, cols);
}
// Grid of M token rows x N output columns in tiles of a short form.
inline TileGrid short_grid(int64_t M, int64_t N, bool gateup, ShortShape f) {
    return spread_tiles(M, N, f.tm, gateup ? f.tn / 2 : f.tn);
}

// Cost of a launch of M token rows, contraction length K, in the tiles f of grid g; < 0: too many tiles.
inline double moved_cost(const TileGrid& g, int64_t M, int64_t K, bool gateup, ShortShape f, int cus) {
    const uint32_t cols = gateup ? f.tn / 2 : f.tn;
    if (g.tiles > (uint64_t)kMaxTiles) return -1;
    const uint32_t tiles = (uint32_t)g.tiles, full = tiles / cus, rem = tiles % cus, rounds = full + (rem ? 1 : 0);
    // a last round on few CUs moves its operands a little faster (3584 / 16 = 224 of 256 CUs: 0.94)
    const double moved = (K < kLongK || !rem) ? rounds : full + 0.85 + 0.15 * rem / cus;
    // Operand rows of a tile, averaged over the token tiles.  Where the last token tile of each group is clearly
    // shorter, a launch of one round is faster than its rows say: the CUs of that tile run ahead of the
    // others and bring the weights into the L2 for them (512 rows in tiles of 160, 160, 160, 32 x 64:
    // 83 us, in four of 128 x 64: 94 us; 1024 rows in two such groups x 128: 126 us, in eight of 128 x 128:
    // 132 us, both over many passes; one pass at a time 116 and 134).  Larger tiles, which wait less for their operands, gain nothing (1280 rows in tiles of 192 x 128,
    // the last of each group 64: 154 us, in eight of 160: 149 us).
    double rows = (double)M / g.tiles_m + f.tn;
    const int last = (int)(g.group_rows - (g.per_group - 1) * f.tm);
    if (K >= kLongK && rounds == 1 && g.per_group > 1 && f.tm * f.tn <= 160 * 128)
        rows *= 10 * last <= 4 * f.tm ? (f.tm * f.tn > 96 * 128 ? 0.92 : 0.87) : 10 * last <= 7 * f.tm ? 0.94 : 1.0;
    const double fixed = kTileFixed + f.tm * cols * (gateup ? kTileFixedPerGateUp : kTileFixedPerDown);
    // (with a long contraction a second workgroup on the CU only shares its loads in flight: 1 row of gate/up in 448
    // tiles of 64 x 64 48 us, in 224 of 64 x 128 43 us)
    const uint32_t together = K < kLongK ? f.per_cu : 1;
    return moved * rows * K + (rounds + together - 1) / together * fixed;
}

// Whether a gate/up launch reads its weights by non-temporal loads: where one group of token tiles covers
// all rows, so that the fabric is asked for every weight line once, and the weights of the layer (half as
// much again for the down projection) are more than the Infinity Cache holds.  Then W_down stays there from
// mini-sequence to mini-sequence instead of being displaced each time, and the stream itself is faster.
// Measured, gate/up and down: 16 rows 43.2 -> 41.8 us and 27.3 (first use, as before), Qwen-shaped 61 rows 54.7 ->
// 51.5, mini-sequences of 512 rows 91.2 + 83.4 -> 87.3 + 79.8, of 1024 rows 162.4 + 122.6 -> 161.0 + 114.1.  With
// four groups (4096 rows) the other groups miss what the first had brought: 615 -> 635 us, so not there; and where
// there is only one mini-sequence, only for at most two token tiles (1000 rows: 161.6 -> 163.9 us).
// The down projection itself loses with it wherever tiles share a weight line: 61 rows 39 -> 51 us.
inline bool weights_once(int64_t tiles_m, int64_t N, int64_t K, bool more_mini_sequences) {
    return tiles_m <= (more_mini_sequences ? kTokenGroup : 2) && 6 * N * K > ((int64_t)256 << 20);
}

// The short form with the least cost; its cost in `cost`; -1: none.
inline int choose_short_form(int64_t M, int64_t N, int64_t K, bool gateup, int cus, double& cost) {
    int best = -1;
    for (int i = 0; i < short_forms(gateup); ++i) {
        const ShortShape f = short_shape(gateup, i);
        const double c = moved_cost(short_grid(M, N, gateup, f), M, K, gateup, f, cus);
        if (c >= 0 && (best < 0 || c < cost)) { best = i; cost = c; }
    }
    return best;
}

// How a launch runs.  All forms give identical bits (every output element sees the same MFMA sequence over k), so
// the choice is free.
enum LaunchKind {
    kRefused,        // too many tiles for 32-bit tile numbers
    kShortTiles,     // gemm_short_kernel, form `form`
    kWholeTiles,     // gemm4_kernel: tiles of tm token rows x tn staged weight rows
    kTwoWidths       // gemm4_two_width_kernel: columns [0, wide_cols) in 256 x 256 tiles (`grid`), the rest in 256 x 192 (`narrow`)
};
struct Launch {
    LaunchKind kind;
    int form, tm, tn;
    int64_t wide_cols;
    TileGrid grid, narrow;
};
inline Launch short_launch(int64_t M, int64_t N, bool gateup, int form) {
    const ShortShape f = short_shape(gateup, form);
    const TileGrid g = short_grid(M, N, gateup, f);
    return {g.tiles > 0 && g.tiles <= (uint64_t)kMaxTiles ? kShortTiles : kRefused, form, f.tm, f.tn, 0, g, {}};
}
inline Launch whole_launch(int64_t M, int64_t N, bool gateup, int tm, int tn) {
    const TileGrid g = whole_tiles(M, N, tm, gateup ? tn / 2 : tn);
    return {g.tiles > 0 && g.tiles <= (uint64_t)kMaxTiles ? kWholeTiles : kRefused, 0, tm, tn, 0, g, {}};
}

// Gate/up tiles of 96 columns beside those of 128: a column of the narrow tile costs 7 % more (measured over
// whole rounds), and the mix has to save this much of the modelled time before it is used.
constexpr int kGateUpNarrowPerMille = 1070;
constexpr int kGateUpMixMinGainPerMille = 15;
// Weight rows of the 256-row tiles of the down projection, and what a narrower tile costs per column (measured).
constexpr int kDownWidths[5] = {256, 224, 192, 160, 128};
constexpr int kDownWidthPerMille[5] = {1000, 1020, 1070, 1170, 1310};

// Rounds of the CUs a launch of `tiles` 256-row tiles takes, in 1/1000.  A last round that fills only part of the
// CUs is not as dear as a whole one: the chip is power-limited and clocks the busy CUs higher (measured:
// a round on a quarter / half / three quarters of the CUs takes about 0.55 / 0.8 / 0.8-0.9 of a full one).
inline int64_t rounds_per_mille(int64_t tiles, int cus) {
    const int64_t full = tiles / cus, rem = tiles % cus;
    return full * 1000 + (rem ? 500 + 500 * rem / cus : 0);
}
// The cost of 256-row tiles that the matrix cores bound, in the units of the short forms: c = rounds x columns in 1e-6.
inline double full_cost(int64_t c, int64_t tiles, int64_t K, bool gateup, int cus) {
    return 1e-6 * c / (gateup ? 128 : 256) * kFullTileRows * K + (tiles + cus - 1) / cus * kFullTileFixed;
}
// ... of the down projection in tiles w weight rows wide; a narrow one is bound by its operands, too (1536 rows x
// 3584 columns: 233 us in tiles 128 wide).
inline double whole_down_cost(int64_t M, int64_t N, int64_t K, int w, int64_t c, int cus) {
    const TileGrid g = whole_tiles(M, N, 256, w);
    const double moved = moved_cost(g, M, K, false, {256, w, 1}, cus), full = full_cost(c, (int64_t)g.tiles, K, false, cus);
    return full > moved ? full : moved;
}

// Down projection with 256-row tiles: 256, 224, 192, 160 or 128 weight rows per tile, whichever needs the least time
// in rounds of the CUs (rounds x width, a narrower tile charged more per column for the token fragments it shares
// among fewer MFMAs, a partly filled last round less than a whole one): 3584 output columns with 32 token tiles are
// 1.75 rounds of 256-wide tiles on 256 CUs but exactly 2 rounds of 224-wide ones, and the 128 full-size tiles of a
// 2048-row mini-sequence at 4096 columns are one round of 256 tiles 128 wide.
// Few tiles: the short forms where their cost is lower.  Then the operand rows that a CU moves count, and the best
// form is the one that gives every CU one tile with the fewest of them.
// Both sides are priced on the grid that runs: 2400 rows x 4096 columns are 220 tiles of 256 x 192 = one round, 223 us,
// against two rounds of 160 x 128, 276 us (2700 rows 231 and 302, 4300 402 and 463, 5500 461 and 595 us).
// full_tiles: tiles of 256 x 256 however few (beside a gate/up kernel that fills the chip).
inline Launch choose_down(int64_t M, int64_t N, int64_t K, int cus, bool full_tiles) {
    if (whole_tiles(M, N, 256, 256).tiles > (uint64_t)kMaxTiles) return {kRefused, 0, 0, 0, 0, {}, {}};
    if (full_tiles) return whole_launch(M, N, false, 256, 256);
    int width = 0;
    int64_t cost = 0;                    // rounds x columns of 256 x 256 tiles, in 1e-6
    for (int i = 0; i < 5; ++i) {
        const int w = kDownWidths[i];
        const int64_t c = rounds_per_mille((int64_t)whole_tiles(M, N, 256, w).tiles, cus) * w * kDownWidthPerMille[i];
        if (width == 0 || c < cost) { cost = c; width = w; }
    }
    double least = 0;
    const int form = choose_short_form(M, N, K, false, cus, least);
    if (form >= 0 && least < whole_down_cost(M, N, K, width, cost, cus)) return short_launch(M, N, false, form);
    return whole_launch(M, N, false, 256, width);
}

// Gate/up with 256-row tiles: the first columns in tiles of 128 columns, the rest in tiles of 96, in one launch of
// the two-width kernel, where the same model says that saves time: 14336 columns with 12 token tiles are 1344 tiles
// = 5.25 rounds, but 64 x 128 + 64 x 96 columns are three rounds of each width.
// Few tiles: the short forms, as for the down projection.  A short contraction: 128-row tiles, two workgroups per CU,
// by the same cost.
inline Launch choose_gateup(int64_t M, int64_t N, int64_t K, int cus) {
    const Launch plain_launch = whole_launch(M, N, true, 256, 256);
    if (plain_launch.kind == kRefused) return plain_launch;
    double least = 0;
    const int form = choose_short_form(M, N, K, true, cus, least);
    // b column tiles of 96 behind a of 128: a = ceil((N - 96 b) / 128); time = rounds x columns per tile
    const int64_t tm = plain_launch.grid.tiles_m;
    auto mix_cost = [&](int64_t b) {
        const int64_t rest = N - 96 * b, wide = rest > 0 ? (rest + 127) / 128 : 0;
        return rounds_per_mille(tm * wide, cus) * 128 * 1000 + rounds_per_mille(tm * b, cus) * 96 * kGateUpNarrowPerMille;
    };
    const int64_t plain = mix_cost(0);
    int64_t cost = plain, narrow_tiles_n = 0;
    // (no mix takes less than half of what the plain tiles take: where the short form does, it is not looked for)
    const bool few = form >= 0 && least < 0.5 * full_cost(plain, 1, K, true, cus);
    for (int64_t b = 1; b <= (N + 95) / 96 && !few; ++b) {
        const int64_t c = mix_cost(b);
        if (c < cost && c * 1000 <= plain * (1000 - kGateUpMixMinGainPerMille)) { cost = c; narrow_tiles_n = b; }
    }
    if (form >= 0) {
        const double full = full_cost(cost, (int64_t)plain_launch.grid.tiles, K, true, cus);
        const Launch whole128 = whole_launch(M, N, true, 128, 128);
        const double cost128 = moved_cost(whole128.grid, M, K, true, {128, 128, 2}, cus);
        if (cost128 >= 0 && cost128 < full && cost128 < least) return whole128;
        if (least < full) return short_launch(M, N, true, form);
    }
    const int64_t rest = N - 96 * narrow_tiles_n, wide_cols = rest > 0 ? (rest + 127) / 128 * 128 : 0;
    if (narrow_tiles_n == 0 || wide_cols >= N) return plain_launch;
    if (wide_cols == 0) return whole_launch(M, N, true, 256, 192);
    Launch l = {kTwoWidths, 0, 256, 256, wide_cols, whole_tiles(M, wide_cols, 256, 128), whole_tiles(M, N - wide_cols, 256, 96)};
    if (l.grid.tiles > (uint64_t)kMaxTiles || l.narrow.tiles > (uint64_t)kMaxTiles) l.kind = kRefused;
    return l;
}

}  // namespace momk

#endif  // MOM_GEMM_FORMS_H

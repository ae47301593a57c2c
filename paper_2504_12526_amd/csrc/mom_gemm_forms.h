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

// Token tiles of a launch: groups of at most kTokenGroup tiles (their weights are fetched by one XCD at a time), the
// rows spread evenly over the groups.
constexpr int kTokenGroup = 4;
// (32-bit arithmetic: every launch walks all forms on the host, and M + 1024 < 2^32.)
struct TokenTiles { uint32_t groups, group_rows, per_group, tiles; };
inline TokenTiles token_tiles(int64_t rows, uint32_t tm) {
    const uint32_t M = (uint32_t)rows, most = kTokenGroup * tm;
    TokenTiles t = {1, M, (M + tm - 1) / tm, 0};
    if (M > most) {
        t.groups = (M + most - 1) / most;
        t.group_rows = (M + t.groups - 1) / t.groups;
        t.groups = (M + t.group_rows - 1) / t.group_rows;
        t.per_group = (t.group_rows + tm - 1) / tm;
    }
    t.tiles = (t.groups - 1) * t.per_group + (M - (t.groups - 1) * t.group_rows + tm - 1) / tm;
    return t;
}

// Cost of a launch of M token rows x N output columns, contraction length K, in tiles of form f; < 0: too many tiles.
inline double short_cost(int64_t M, int64_t N, int64_t K, bool gateup, ShortShape f, int cus) {
    const uint32_t cols = gateup ? f.tn / 2 : f.tn;
    const TokenTiles t = token_tiles(M, f.tm);
    const uint64_t all = (uint64_t)t.tiles * (((uint32_t)N + cols - 1) / cols);
    if (all > (uint64_t)kMaxTiles) return -1;
    const uint32_t tiles = (uint32_t)all, full = tiles / cus, rem = tiles % cus, rounds = full + (rem ? 1 : 0);
    // a last round on few CUs moves its operands a little faster (3584 / 16 = 224 of 256 CUs: 0.94)
    const double moved = (K < kLongK || !rem) ? rounds : full + 0.85 + 0.15 * rem / cus;
    // Operand rows of a tile, averaged over the token tiles.  Where the last token tile of each group is clearly
    // shorter, a launch of one round is faster than its rows say: the CUs of that tile run ahead of the
    // others and bring the weights into the L2 for them (512 rows in tiles of 160, 160, 160, 32 x 64:
    // 83 us, in four of 128 x 64: 94 us; 1024 rows in two such groups x 128: 126 us, in eight of 128 x 128:
    // 132 us, both over many passes; one pass at a time 116 and 134).  Larger tiles, which wait less for their operands, gain nothing (1280 rows in tiles of 192 x 128,
    // the last of each group 64: 154 us, in eight of 160: 149 us).
    double rows = (double)M / t.tiles + f.tn;
    const int last = (int)(t.group_rows - (t.per_group - 1) * f.tm);
    if (K >= kLongK && rounds == 1 && t.per_group > 1 && f.tm * f.tn <= 160 * 128)
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

// The form with the least cost; its cost in `cost`; -1: none.
inline int choose_short_form(int64_t M, int64_t N, int64_t K, bool gateup, int cus, double& cost) {
    int best = -1;
    for (int i = 0; i < short_forms(gateup); ++i) {
        const double c = short_cost(M, N, K, gateup, short_shape(gateup, i), cus);
        if (c >= 0 && (best < 0 || c < cost)) { best = i; cost = c; }
    }
    return best;
}

}  // namespace momk

#endif  // MOM_GEMM_FORMS_H

// Tile forms of the GEMM launches with few token rows, and the rule that picks one.  Plain C++17, no HIP
// types, so that a host program can walk the rule (tests/gemm_forms_check.cpp).
//
// X(TM, TN, WM, WN, KSUB, NSTG): TM token rows x TN staged weight rows per workgroup, WM x WN wavefronts
// that multiply, stages of 64 KSUB K-elements, NSTG of them in the LDS ring (mom_gemm_short.hip.inc).
// The smallest tiles take the longest stages (one barrier per stage) and nearly every form a ring that holds
// more than the 32 KiB a CU's vector cache has in flight at most (measured: 256 lines of 128 bytes).  Gate/up
// 64 x 64 has two rings: of three slots, so that three workgroups fit a CU (33 rows of H = 8192, I = 28672: 155 us, with five
// slots 187), and of five for launches that give a CU only one (the same rows at I = 3584: 51 us, with five slots 36).
#ifndef MOM_GEMM_FORMS_H
#define MOM_GEMM_FORMS_H

#include <stdint.h>

#include <initializer_list>

#define MOM_SHORT_FORMS_DOWN(X)                                                                          \
    X(16, 16, 1, 1, 2, 8) X(32, 16, 2, 1, 4, 6) X(32, 32, 2, 2, 2, 5) X(48, 32, 1, 2, 2, 8)              \
    X(64, 32, 2, 2, 2, 6) X(96, 32, 2, 2, 2, 5) X(32, 64, 2, 2, 1, 6) X(64, 64, 2, 2, 1, 5)              \
    X(80, 64, 1, 4, 2, 4) X(96, 64, 2, 2, 2, 4) X(128, 64, 2, 2, 1, 6) X(160, 64, 2, 2, 1, 5)            \
    X(192, 64, 2, 2, 1, 5) X(256, 64, 2, 2, 1, 4) X(96, 128, 2, 2, 1, 5) X(128, 128, 2, 2, 1, 5)         \
    X(160, 128, 2, 2, 1, 4) X(192, 128, 2, 2, 1, 4) X(224, 128, 2, 2, 1, 3)                              \
    X(32, 48, 2, 1, 2, 8) X(48, 48, 3, 1, 2, 6) X(64, 48, 4, 1, 2, 5) X(80, 48, 1, 3, 2, 5)              \
    X(96, 48, 2, 1, 2, 4) X(80, 32, 1, 2, 2, 5) X(48, 64, 1, 4, 2, 5) X(96, 96, 2, 2, 1, 6)              \
    X(128, 96, 2, 2, 1, 5) X(160, 96, 2, 2, 1, 5)
#define MOM_SHORT_FORMS_GATEUP(X)                                                                        \
    X(16, 32, 1, 1, 4, 6) X(32, 32, 2, 1, 2, 8) X(16, 64, 1, 2, 2, 8) X(32, 64, 2, 2, 2, 6)              \
    X(64, 64, 2, 2, 1, 3) X(128, 64, 2, 2, 1, 3) X(64, 128, 2, 2, 1, 6) X(96, 128, 2, 2, 1, 5)           \
    X(128, 128, 2, 2, 1, 5) X(160, 128, 2, 2, 1, 4) X(192, 128, 2, 2, 1, 4) X(224, 128, 2, 2, 1, 3)      \
    X(64, 192, 2, 2, 1, 5) X(96, 192, 2, 2, 1, 4) X(128, 192, 2, 2, 1, 4) X(64, 64, 2, 2, 1, 5)

// X(TM, TN) of the rectangular tiles (mom_gemm_rect.hip.inc): those of 54 measured that are the best of some launch by more
// than the next.
#define MOM_RECT_FORMS_DOWN(X)                                                                           \
    X(160, 160) X(160, 256) X(192, 160) X(192, 224) X(192, 256) X(224, 160) X(224, 224) X(224, 256)
#define MOM_RECT_FORMS_GATEUP(X)                                                                         \
    X(256, 128) X(160, 160) X(192, 160) X(224, 160) X(256, 160) X(320, 160) X(288, 192) X(320, 192)      \
    X(160, 224) X(192, 224) X(256, 224) X(288, 224) X(224, 256) X(192, 320)                              \
    X(96, 160) X(128, 160) X(96, 224) X(128, 224)

namespace momk {

// per_cu: workgroups that a CU's 160 KiB of LDS hold; ahead: K-elements that a workgroup has in flight at most.
struct ShortShape { int tm, tn, per_cu, ahead; };
#define MOM_SHAPE(TM, TN, WM, WN, KSUB, NSTG) \
    {TM, TN, 163840 / (NSTG * KSUB * (TM + TN) * 128) > 4 ? 4 : 163840 / (NSTG * KSUB * (TM + TN) * 128), (NSTG - 1) * 64 * KSUB},
constexpr ShortShape kShortDown[] = {MOM_SHORT_FORMS_DOWN(MOM_SHAPE)};
constexpr ShortShape kShortGateUp[] = {MOM_SHORT_FORMS_GATEUP(MOM_SHAPE)};
#undef MOM_SHAPE
constexpr int kShortDownForms = sizeof(kShortDown) / sizeof(kShortDown[0]);
constexpr int kShortGateUpForms = sizeof(kShortGateUp) / sizeof(kShortGateUp[0]);

// Down forms that are looked at for layers that stay in the Infinity Cache: the later ones gain nothing there (their launches take 5
// ... 20 us, and the formula's best of them 0.4 % more on average).
constexpr int kSmallDownForms = 19;
inline int short_forms(bool gateup) { return gateup ? kShortGateUpForms : kShortDownForms; }
inline ShortShape short_shape(bool gateup, int form) { return gateup ? kShortGateUp[form] : kShortDown[form]; }

// Index of the (first) form with these tiles, or -1.
inline int find_short_form(bool gateup, int tm, int tn) {
    for (int i = 0; i < short_forms(gateup); ++i)
        if (short_shape(gateup, i).tm == tm && short_shape(gateup, i).tn == tn) return i;
    return -1;
}

// Rectangular tiles, by their sizes: one workgroup per CU.
#define MOM_SHAPE(TM, TN) {TM, TN, 1, 0},
constexpr ShortShape kRectDown[] = {MOM_RECT_FORMS_DOWN(MOM_SHAPE)};
constexpr ShortShape kRectGateUp[] = {MOM_RECT_FORMS_GATEUP(MOM_SHAPE)};
#undef MOM_SHAPE
constexpr int kRectDownForms = sizeof(kRectDown) / sizeof(kRectDown[0]);
constexpr int kRectGateUpForms = sizeof(kRectGateUp) / sizeof(kRectGateUp[0]);
inline int rect_forms(bool gateup) { return gateup ? kRectGateUpForms : kRectDownForms; }
inline ShortShape rect_shape(bool gateup, int form) { return gateup ? kRectGateUp[form] : kRectDown[form]; }
inline bool is_rect_form(bool gateup, int tm, int tn) {
    for (int i = 0; i < rect_forms(gateup); ++i)
        if (rect_shape(gateup, i).tm == tm && rect_shape(gateup, i).tn == tn) return true;
    return false;
}

constexpr int64_t kMaxTiles = 0x1fffffff;            // tile numbers are 32-bit in the kernels

// The tiles of a launch, as it is priced AND as it is launched: tiles_m token tiles one after the other, walked in groups
// of kTokenGroup (their weights are fetched by one XCD at a time), tiles_n column tiles.
// (32-bit arithmetic: every launch walks all forms on the host, and M + 1024 < 2^32.)
constexpr int kTokenGroup = 4;
struct TileGrid { uint32_t tiles_m, tiles_n; uint64_t tiles; };
inline TileGrid tile_grid(int64_t M, int64_t N, bool gateup, ShortShape f) {
    const uint32_t cols = gateup ? f.tn / 2 : f.tn;
    const uint32_t tm = ((uint32_t)M + f.tm - 1) / f.tm, tn = ((uint32_t)N + cols - 1) / cols;
    return {tm, tn, (uint64_t)tm * tn};
}

// Tile number of workgroup bid.  Workgroup ids go round-robin over the 8 XCDs: each gets a contiguous run of tile numbers
// (tiles_per_xcd of them; those past the last tile have nothing to do).
constexpr int tiles_per_xcd(uint64_t tiles) { return (int)((tiles + 7) / 8); }
constexpr int tile_number(int bid, int tiles_per_xcd) { return (bid & 7) * tiles_per_xcd + (bid >> 3); }

// Where tile number vt lies: groups of group_m token tiles one after the other, in a group the token tiles of one column
// tile first.
struct TilePlace { int m, n; };
constexpr TilePlace tile_place(int vt, int tiles_m, int tiles_n, int group_m) {
    const int per_group = group_m * tiles_n;
    const int grp = vt / per_group;
    const int first_m = grp * group_m;
    const int gsz = tiles_m - first_m < group_m ? tiles_m - first_m : group_m;
    const int in_grp = vt - grp * per_group;
    return {first_m + in_grp % gsz, in_grp / gsz};
}

// What ring load j of a wavefront of a short form moves in each stage: 8 rows of 64 K-elements, from sub-tile sub and row
// src on of its operand (of W_gate or W_up, for gate/up) to row `row` of the operand tile.  The tokens' LT loads come first.
struct RingLoad { bool token; int sub, row, src; };
constexpr RingLoad ring_load(bool gateup, int TM, int TN, int KSUB, int wave, int j) {
    const int LT = KSUB * TM / 32;
    if (j < LT) {
        const int b = wave + 4 * j, row = (b % (TM / 8)) * 8;
        return {true, b / (TM / 8), row, row};
    }
    const int HR = gateup ? TN / 2 : TN;                                // rows of one weight matrix
    const int w = wave + 4 * (j - LT);
    const int half = w / (KSUB * HR / 8), b = w % (KSUB * HR / 8);
    const int src = (b % (HR / 8)) * 8;
    return {false, b / (HR / 8), half * HR + src, src};
}
// Whether weight load j reads W_up, whichever wavefront it is (gate/up).
constexpr bool ring_load_up(int TM, int TN, int KSUB, int j) { return j - KSUB * TM / 32 >= KSUB * TN / 64; }

// In which order the stages of a short form's ring (nstg of them, `loads` loads per wavefront and stage) are requested, and what the kernel waits
// for.  Stage 0 ... nstg - 1 before the first is multiplied, then, while stage t is and the last of its group by place is done, those of the next group:
// `group` stages together, load by load, one behind the other.  Group boundaries lie so that the stages in front of nstg end one.
//   ring_place       place of stage t in its group
//   ring_first       the first stage that is requested while stage t is multiplied, and group - 1 behind it; -1: none.  All go to slots (stage %
//                    nstg) of stages up to t, which are in registers.
//   ring_in_flight   loads that may still be on their way when stage t is needed and `ahead` stages are requested behind it
constexpr int ring_place(int t, int nstg, int group) { return ((t - nstg) % group + group) % group; }
constexpr int ring_first(int t, int nstg, int group) { return t % group == group - 1 ? t + nstg - group + 1 : -1; }
constexpr int ring_in_flight(int t, int ahead, int nstg, int group, int loads) {
    const int r = group - 1 - ring_place(t, nstg, group), n = r + (ahead - r) * loads;
    return n > 63 ? 63 : n;
}
// ... when stage t + 1 is needed at the barrier of stage t: that many stages are requested behind it.
constexpr int ring_ahead(int t, int nstg, int group) { return nstg - 2 - t % group; }

// The time of a launch in us: what a CU spends on a tile, times the tiles it runs.
//   start, output   once per tile: launch, ring prologue, epilogue; per output element (silu for gate/up).  The workgroups
//                   that share a CU (ShortShape::per_cu) overlap it.
//   row, fetched    per K-element: the operand rows that the CU moves into its LDS, and its share of the rows that its XCD
//                   fetches from beyond the L2.  A CU's vector cache has 256 lines in flight, and at the latency of weights
//                   that come from HBM that is 55 GB/s, whatever the ring holds and however little is multiplied; rows
//                   that another CU of the XCD has fetched before cost about a third of that.
//   product         per K-element: token rows x weight rows, the matrix cores.
//   last_round      a last round on few CUs takes this much of a whole one, and the rest in proportion: the
//                   chip is power-limited and clocks the busy CUs higher.
//   latency         a workgroup waits at least this long for what it has in flight (ShortShape::ahead): 0.69 us from HBM,
//                   0.33 us from the Infinity Cache.
//   whole_tile      the token rows are those of a whole tile, which the launch waits for; otherwise those of an average one.
//   lead            the part per K-element is less by this and by lead_small x 64 / (tm + tn) where the last token tile has
//                   clearly fewer rows, the launch is one round and W_down at most lead_mib: the CUs of that tile run
//                   ahead and bring the weights nearer for the others, less so in tiles below 48 rows (1000 rows x 4096 columns in tiles of 160, six of them
//                   and one of 40, x 128: 119 us; as eight even ones of 128: 133 us; 512 rows x 5120 columns, K = 25600, in
//                   160 x 96 166 us, in 128 x 96 200 us).
//   lead_few        above four token tiles less the more there are: the CUs ahead are fewer of all (512 rows as above in
//                   96 x 128, five and a third: 192 us); and less in tiles above 160 x 128.
// Fitted to every form on 1 ... 4096 rows of eleven layers (H 256 ... 8192, I 1024 ... 28672), single calls and loops of
// mini-sequences.  Formula and time of the forms near the best of their size differ by 5 (256-row tiles), 8 (short, down)
// and 9 % (short, gate/up; the least of many uncertain times is an optimistic one, so these figures are the fitted ones
// and 5 or 6 % on everything).  Over the 1427 launches measured, the form of least time takes 1 % longer than the best of
// all forms on average, and more than 10 % longer in 22 of them; in the down projection of six layers with 48 other row
// counts from 258 to 2440, 1.1 % and in 6 of 288.
struct LaunchTime {
    double start, output, row, fetched, product, last_round, latency;
    bool whole_tile;
    double lead, lead_small;
    int lead_mib = 160;
    bool lead_few = false;
};
constexpr double kFromHbm = 0.69, kFromCache = 0.33;
// Down, weights from HBM and (kShortDownKeptTime) from the Infinity Cache: by what the choice costs, on 59 row counts from 1 to 2048
// of six layers (H 2048 ... 8192), launches of one form after the other: 0.5 % (236 launches, none above 10 %) and 0.6 % (177, 2 above
// 10 %) over the best of 37 forms; with the 20 forms and the constants before, 2.5 % (29) and 2.2 % (28).  Inside calls, behind a
// gate/up launch and with weights not used before, on 40 ... 1900 rows of ten layers (H 3584 ... 8192) with W_down of up to 470 MB:
// 0.7 % (179 launches, 2 above 10 %); without lead_mib, lead_few and kOverWhole 3.0 % (20).  kShortDownTime is fitted again to whole
// calls: 882 of 16 ... 990 rows of 14 layers (H 2048 ... 8192, weights from HBM), all forms near the best of each forced in turn.  The
// calls take 0.38 % more than with the best form, 5 of them above 6 %; before, 0.47 % and 13, because the lead of small tiles was
// overrated: 57 ... 64 rows x 2048 columns, K = 8192, as 128 tiles of 48 x 32 (calls of 36.0 us) instead of 256 of 32 x 16 (32.9), 86
// rows as 128 of 64 x 32 (40.1) instead of 192 of 32 x 32 (37.4).  From long_from rows on, where
// it is the 256-row and rectangular tiles that a short form is compared with, kShortDownLongTime, fitted together with those (1536
// rows x 4096 columns in 192 x 128: 160 us, so 159, by kShortDownTime 178).
constexpr LaunchTime kShortDownTime = {5.46, 2.25e-5, 2.20e-5, 5.11e-5, 7.76e-8, 1.0, kFromHbm, true, 0.212, 0.0855, 256, true};
constexpr LaunchTime kShortDownLongTime = {4.0, 5.0e-5, 1.94e-5, 5.56e-5, 5.81e-8, 1.0, kFromHbm, true, 0.1, 0.2};
constexpr LaunchTime kShortDownKeptTime = {2.28, 9.78e-5, 1.14e-5, 4.14e-5, 7.43e-8, 1.0, kFromCache, true, 0, 0};
// W_down still in the Infinity Cache.  Then nobody needs to run ahead: 1024 rows x 4096 columns in tiles of
// 160 x 128: 117 us, in eight of 128 x 128: 109 us; 512 rows in tiles of 160 x 64 80 us, of 128 x 64 70 us.
constexpr LaunchTime kShortDownSmallTime = {5.9, 1.40e-4, 1.02e-5, 3.58e-5, 1.36e-7, 1.0, kFromCache, true, 0, 0};
// (Gate/up: fitted before rings of five stages and more requested two together.  Those with weights from memory take less than the formula
// where K is a multiple of 4096: 96 rows x 14336 columns, K = 4096, 47 us, 51 by the formula, 128 rows 50 and 55.)
constexpr LaunchTime kShortGateUpTime = {5.95, 1.97e-4, 1.11e-5, 5.61e-5, 1.42e-7, 1.0, kFromHbm, false, 0, 0};
constexpr LaunchTime kShortGateUpSmallTime = {6.15, 2.28e-4, 1.20e-5, 3.92e-5, 1.41e-7, 1.0, kFromCache, false, 0, 0};
constexpr LaunchTime kFullDownTime = {4.0, 2.4e-5, 1.09e-5, 4.87e-5, 1.52e-7, 0.80, 0, true, 0, 0};
constexpr LaunchTime kFullGateUpTime = {4.0, 1.90e-4, 7.3e-6, 2.63e-5, 2.04e-7, 0.72, 0, true, 0, 0};
// The 128-row gate/up tiles of mom_gemm.hip.inc, two workgroups per CU, a ring of 2.5 stages each of which about one is in
// flight: one 128 x 128 tile per CU at K = 8192 takes 95 us, in the short form 59 us.  They are looked at for launches of up
// to two rounds with a short contraction, and of one to two rounds in several groups of token tiles: two rounds at K = 1024
// 20.4 us, 1.75 rounds at K = 8192 in two groups 110 us, against 22.5 and 116 us in the best other form; but 1.75 rounds
// at K = 4096 in one group 82 us against 73, and 4.6 rounds at K = 3584 190 us against 124.
constexpr LaunchTime kPairGateUpTime = {6.6, 9.6e-5, 2.65e-5, 0, 0, 1.0, kFromHbm, false, 0, 0};
constexpr LaunchTime kPairGateUpSmallTime = {6.6, 9.6e-5, 2.65e-5, 0, 0, 1.0, kFromCache, false, 0, 0};
constexpr ShortShape kPairShape = {128, 128, 2, 58};
// Rectangular tiles, fitted to 54 forms of them, those near the best of a launch weighted most: gate/up to 100 ... 16384 rows of
// four layers above 128 MiB (H 3584 ... 8192; formula and time differ by 4 %), down to 1000 ... 16384 rows of the same (4 %, and the
// forms by what kRectDownPerMille says).  Times of launches one after the other; between calls that alternate, the two-width and 256 x 256
// gate/up launches gain 2-5 % on them.  So a rectangular tile has to promise more than the others' formula by the share given:
// kOverOneRound   gate/up, 256 x 256 tiles of more than one round: at 0.945 ... 0.975 promised 0.95 ... 1.06 of the time came
//                 (1000 rows x 18944 columns 0.964: 203 -> 212 us), below mostly as promised (850 rows 0.74: 198 -> 161 us)
// kOneTokenTile   gate/up, 256 x 256 tiles of up to 256 rows: 17920 columns, K = 5120, 256 rows 101 -> 93 us, promised 0.9 ... 1.03
// kOverShort      gate/up short forms, whose time at 97 ... 224 rows is overrated: 0.83 ... 0.90 promised 0.97 ... 1.0
// kOverShortFilled  the same at 24 ... 128 rows where one token tile of them keeps 7/8 of the CUs busy or more, and no less than
//                 the weights take at 5.6 TB/s: 18944 columns, K = 3584, 64 rows 51.4 -> 47.8 us, 25600, K = 5120, 119.7 ->
//                 94.5; on 180 of 256 CUs (14336 columns, K = 4096) they lose (96 rows 45.7 -> 50.5)
// kOverDown       down, either kind, after the correction: 2900 rows x 4096 columns 0.89 promised, 247 -> 233 us
// kOverWhole      down below long_from rows, where the formula underrates the whole tiles against the short ones: 700 rows x 8192
//                 columns, K = 28672, in 192 x 128 325, in 256 x 128 362 us at 344 and 326 promised
constexpr LaunchTime kRectGateUpTime = {3.73, 3.07e-5, 1.09e-5, 4.22e-5, 1.68e-7, 0.74, 0, true, 0, 0};
constexpr LaunchTime kRectDownTime = {7.24, 2.95e-5, 2.34e-5, 7.72e-6, 1.02e-7, 0.707, 0, true, 0.048, 0};
constexpr int kRectDownPerMille[kRectDownForms] = {1000, 970, 970, 975, 1010, 960, 1010, 1040};
constexpr double kOverOneRound = 0.945, kWithinOneRound = 0.975, kOneTokenTile = 1.03;
constexpr double kOverShort = 0.83, kOverShortFilled = 0.975, kOverDown = 0.975, kOverWhole = 0.9;
constexpr double kRectBytes = 4 / 5.6e6;        // us per weight pair at 5.6 TB/s

// Whether weight rows x K of them leave the Infinity Cache room (192 MiB do: 6144 columns, K = 16384, in mini-sequences of 256 rows
// 1154 us in the tiles for weights from HBM, 1047 in those for kept ones; 250 MiB don't, 512 rows x 5120 columns, K = 25600, 4 ... 8 %).
inline bool weights_fit(int64_t rows, int64_t K) { return 2 * rows * K <= ((int64_t)200 << 20); }

// Token rows from which the down projection of N columns is priced by kShortDownLongTime.  Up to 192 MiB of W_down both sets choose as well
// from 1100 to 1300 rows, and at 1150 the same form in every one of 13 layers; with the line at 1000 the form changed for the worse in
// two of them (1004 rows x 6144 columns, K = 16384, calls of 482 us, now 462; x 2560, K = 9728, 160, 155).  From 250 MiB on it changes
// for the better there (1005 rows x 5120 columns, K = 25600, 651, by the other set 660).
inline int64_t long_from(int64_t N, int64_t K) { return weights_fit(N, K) ? 1150 : 1000; }

// A layer that stays in the Infinity Cache between calls (tests, small models): a quarter of it.
inline bool small_layer(int64_t N, int64_t K) { return 6 * N * K <= ((int64_t)64 << 20); }

// A launch of M token rows, contraction length K, in the tiles f of grid g; < 0: too many tiles.
inline double launch_time(const TileGrid& g, int64_t M, int64_t K, bool gateup, ShortShape f, const LaunchTime& t, int cus) {
    if (g.tiles > (uint64_t)kMaxTiles) return -1;
    const uint32_t tiles = (uint32_t)g.tiles, full = tiles / cus, rem = tiles % cus, rounds = full + (rem ? 1 : 0);
    const double moved = full + (rem ? t.last_round + (1 - t.last_round) * rem / cus : 0);
    const double token_rows = (double)M / g.tiles_m;       // of an average tile
    // of a round, an XCD (an eighth of the CUs) runs this many tiles: a group of token tiles by so many weight tiles
    const uint32_t on_xcd = ((full ? (uint32_t)cus : rem) + 7) / 8, group = g.tiles_m < kTokenGroup ? g.tiles_m : kTokenGroup;
    const double fetched = (group * token_rows + (on_xcd + group - 1) / group * f.tn) * 8 / cus;
    const double tile_rows = t.whole_tile ? f.tm : token_rows;
    double per_k = t.row * (tile_rows + f.tn) + t.fetched * fetched + t.product * tile_rows * f.tn;
    if (t.lead > 0 && rounds == 1 && g.tiles_m > 1 && 2 * g.tiles_n * f.tn * K <= (int64_t)t.lead_mib << 20) {
        const double last = (double)(M - (int64_t)(g.tiles_m - 1) * f.tm) / f.tm;      // of the last token tile
        const double ahead = last < 0.4 ? 1 : last < 0.72 ? (0.72 - last) / 0.32 : 0;
        const double shared = !t.lead_few ? 1 : (g.tiles_m > 4 ? 4.0 / g.tiles_m : 1) * (f.tm * f.tn > 160 * 128 ? 0.8 : 1);
        per_k *= 1 - ahead * (f.tm < 48 ? f.tm / 48.0 : 1) * shared * (t.lead + t.lead_small * 64 / (f.tm + f.tn));
    }
    const double once = t.start + t.output * f.tm * (gateup ? f.tn / 2 : f.tn);
    const double starts = (double)rounds / f.per_cu, body = moved * per_k;
    const double least = (rounds + f.per_cu - 1) / f.per_cu * (f.ahead ? t.latency / f.ahead : 0);
    return (starts > 1 ? starts : 1) * once + K * (body > least ? body : least);
}

// Whether a gate/up launch reads its weights by non-temporal loads: where one group of token tiles covers
// all rows, so that the fabric is asked for every weight line once, and the weights of the layer (half as
// much again for the down projection) are more than the Infinity Cache holds.  Then W_down stays there from
// mini-sequence to mini-sequence instead of being displaced each time, and the stream itself is faster.
// Measured, gate/up and down: 16 rows 43.2 -> 41.8 us and 27.3 (first use, as before), Qwen-shaped 61 rows 54.7 ->
// 51.5, mini-sequences of 512 rows 91.2 + 83.4 -> 87.3 + 79.8, of 1024 rows 162.4 + 122.6 -> 161.0 + 114.1 (down in 160 x 64
// and 160 x 128; the even tiles that W_down in the cache has got since, kept_down, take 70 and 105).  With
// four groups (4096 rows) the other groups miss what the first had brought: 615 -> 635 us, so not there; and where
// there is only one mini-sequence, only for at most two token tiles (1000 rows: 161.6 -> 163.9 us).
// The down projection itself loses with it wherever tiles share a weight line: 61 rows 39 -> 51 us.
inline bool weights_once(int64_t tiles_m, int64_t N, int64_t K, bool more_mini_sequences) {
    return tiles_m <= (more_mini_sequences ? kTokenGroup : 2) && 6 * N * K > ((int64_t)256 << 20);
}

// W_down is taken to be in the Infinity Cache: that of a small layer, and from mini-sequence kKeptFrom of a call on where kept_down.
// Down by mini-sequence, other weights in each call: 512 rows in tiles of 128 x 64 97, 93, 72, 72 ... us (of 160 x 64 92, 92, 91, 91);
// 256 rows in 64 x 64 70, 65, 45, 45 (of 80 x 64 58, 55, 53, 53).
constexpr int kKeptFrom = 2;

// Rows of a mini-sequence whose gate/up launch is to pass W_down by: as many as one group of 256-row token tiles.  Its other forms are
// then those of one group too: six mini-sequences of 768 rows x 11008 columns, K = 4096, in five token tiles of 160 x 224, whose weights
// come through the cache and displace W_down, take 1279 us, in three of 256 x 160 1146.
inline bool to_pass_by(int64_t M, int64_t N, int64_t K, bool more_mini_sequences) {
    return more_mini_sequences && M <= 256 * kTokenGroup && 6 * N * K > ((int64_t)256 << 20) && weights_fit(N, K);
}

// The short form that takes the least time; its time in `least`; -1: none.
inline int choose_short_form(int64_t M, int64_t N, int64_t K, bool gateup, const LaunchTime& time, int cus, double& least, int forms = 0,
                             bool one_group = false) {
    int best = -1;
    for (int i = 0; i < (forms ? forms : short_forms(gateup)); ++i) {
        const ShortShape f = short_shape(gateup, i);
        if (one_group && f.tm * kTokenGroup < M) continue;
        const double t = launch_time(tile_grid(M, N, gateup, f), M, K, gateup, f, time, cus);
        if (t >= 0 && (best < 0 || t < least)) { best = i; least = t; }
    }
    return best;
}

// The rectangular tiles that take the least time; their time in `least`; tm 0: none.
inline ShortShape choose_rect_form(int64_t M, int64_t N, int64_t K, bool gateup, const LaunchTime& time, int cus, double& least,
                                   bool one_group = false) {
    ShortShape best = {0, 0, 1, 0};
    for (int i = 0; i < rect_forms(gateup); ++i) {
        const ShortShape f = rect_shape(gateup, i);
        if (one_group && f.tm * kTokenGroup < M) continue;
        if (gateup && f.tm < 160 && M > 224) continue;         // tiles for one token tile, or two (256 rows x 13824 columns: 82 -> 94 us)
        // 192 x 320, whose weights have two ring slots, for two token tiles at most: 384 rows x 18944 columns, K = 3584, calls of 184 us,
        // 192 against the next form; but 700 ... 768 rows x 9728 0.94 ... 0.97 promised of what 256 x 256 takes, 1.03 ... 1.04 measured
        if (gateup && f.tn == 320 && M > 2 * f.tm) continue;
        const double t = launch_time(tile_grid(M, N, gateup, f), M, K, gateup, f, time, cus);
        if (t >= 0 && (best.tm == 0 || t < least)) { best = f; least = t; }
    }
    return best;
}

// How a launch runs.  All forms give identical bits (every output element sees the same MFMA sequence over k), so
// the choice is free.
enum LaunchKind {
    kRefused,        // no such form, or too many tiles for 32-bit tile numbers
    kShortTiles,     // gemm_short_kernel, form `form`
    kWholeTiles,     // tiles of tm token rows x tn staged weight rows: gemm_rect_kernel for those in its list, else gemm4_kernel
    kTwoWidths       // gemm4_two_width_kernel: columns [0, wide_cols) in 256 x 256 tiles (`grid`), the rest in 256 x 192 (`narrow`)
};
struct Launch {
    LaunchKind kind;
    int form, tm, tn;
    int64_t wide_cols;
    TileGrid grid, narrow;
    double time = 0;         // what the choice expects it to take, us (0: not chosen by time)
};
inline Launch timed(Launch l, double time) {
    l.time = time;
    return l;
}
inline Launch short_launch(int64_t M, int64_t N, bool gateup, int form) {
    if (form < 0 || form >= short_forms(gateup)) return {kRefused, 0, 0, 0, 0, {}, {}};
    const ShortShape f = short_shape(gateup, form);
    const TileGrid g = tile_grid(M, N, gateup, f);
    return {g.tiles > 0 && g.tiles <= (uint64_t)kMaxTiles ? kShortTiles : kRefused, form, f.tm, f.tn, 0, g, {}};
}
inline Launch whole_launch(int64_t M, int64_t N, bool gateup, int tm, int tn) {
    const TileGrid g = tile_grid(M, N, gateup, {tm, tn, 1, 0});
    return {g.tiles > 0 && g.tiles <= (uint64_t)kMaxTiles ? kWholeTiles : kRefused, 0, tm, tn, 0, g, {}};
}

// Whether a mini-sequence of M rows leaves W_down (N x K) in the Infinity Cache for the next one, with the gate/up launch given: where
// the layer fits, or that launch passes it by and it leaves room.  Up to 4096 rows, which the constants for it are fitted to: 6000 rows x
// 2048 columns, K = 8192, ran in 192 x 128 by them, 1762 us per four mini-sequences, and run in 192 x 256, 1656, by the others.
inline bool kept_down(const Launch& gateup, int64_t M, int64_t N, int64_t K) {
    if (M > 4096) return false;
    return 6 * N * K <= ((int64_t)256 << 20) || (weights_once(gateup.grid.tiles_m, K, N, true) && weights_fit(N, K));
}

// Gate/up tiles of 96 columns beside those of 128: a column of the narrow tile costs 7 % more (measured over
// whole rounds), and the mix has to save this much of the modelled time before it is used.
constexpr int kGateUpNarrowPerMille = 1070;
constexpr int kGateUpMixMinGainPerMille = 15;
// Rounds of the CUs a launch of `tiles` 256-row tiles takes, in 1/1000.  A last round that fills only part of the
// CUs is not as dear as a whole one: the chip is power-limited and clocks the busy CUs higher (measured:
// a round on a quarter / half / three quarters of the CUs takes about 0.55 / 0.8 / 0.8-0.9 of a full one).
inline int64_t rounds_per_mille(int64_t tiles, int cus) {
    const int64_t full = tiles / cus, rem = tiles % cus;
    return full * 1000 + (rem ? 500 + 500 * rem / cus : 0);
}

// The number b > 0 of column tiles of 96 behind those of 128 in a launch of N columns and tm token tiles for which the rounds of the CUs
// take the least time and kGateUpMixMinGainPerMille less than for b = 0, and that `cost`; 0: none.  The cost of b: rounds_per_mille(tm * a) * 128 *
// 1000 + rounds_per_mille(tm * b) * 96 * kGateUpNarrowPerMille, a = ceil((N - 96 b) / 128).  Every launch looks at all b (148 of them at
// 14336 columns, 2 us of a choice's 2.7 by divisions), so the rounds are counted on from one b to the next.
struct Rounds {
    uint32_t cus, rem = 0;
    int64_t full = 0;
    explicit Rounds(int n) : cus((uint32_t)n) {}
    Rounds(int n, int64_t tiles) : cus((uint32_t)n), rem((uint32_t)(tiles % n)), full(tiles / n) {}
    void count(const Rounds& o, int times) {                   // times: 1 or -1
        full += times * o.full;
        if (times > 0) { rem += o.rem; if (rem >= cus) { rem -= cus; ++full; } }
        else { if (rem < o.rem) { rem += cus; --full; } rem -= o.rem; }
    }
    int64_t per_mille() const { return full * 1000 + (rem ? 500 + 500 * rem / cus : 0); }
};
inline int64_t narrow_tiles(int64_t N, int64_t tm, int cus, int64_t& cost) {
    int64_t a = (N + 127) / 128, best = 0;
    const Rounds column(cus, tm);
    Rounds wide(cus, tm * a), narrow(cus);
    const int64_t plain = wide.per_mille() * 128 * 1000, most = plain * (1000 - kGateUpMixMinGainPerMille);
    cost = plain;
    for (int64_t b = 1, left = N - 96; b <= (N + 95) / 96; ++b, left -= 96) {
        narrow.count(column, 1);
        while (a > 0 && left <= 128 * (a - 1)) { wide.count(column, -1); --a; }
        const int64_t c = wide.per_mille() * 128 * 1000 + narrow.per_mille() * 96 * kGateUpNarrowPerMille;
        if (c < cost && c * 1000 <= most) { cost = c; best = b; }
    }
    return best;
}
// Down projection: 256-row tiles of 256, 224, 192, 160 or 128 weight rows, or the short forms, whatever takes the least time:
// 3584 output columns with 32 token tiles are 1.75 rounds of 256-wide tiles on 256 CUs but exactly 2 rounds of
// 224-wide ones, and the 128 full-size tiles of a 2048-row mini-sequence at 4096 columns are one round of 256 tiles 128 wide.
// With few token rows the operand rows that a CU moves count, and the best form is the one that gives every CU one
// tile with the fewest of them.
// Both sides are priced on the grid that runs: 2400 rows x 4096 columns are 220 tiles of 256 x 192 = one round, 223 us,
// against two rounds of 160 x 128, 276 us (2700 rows 231 and 302, 4300 402 and 463, 5500 461 and 595 us).
// kept: W_down is in the Infinity Cache (kept_down).
inline Launch choose_down(int64_t M, int64_t N, int64_t K, int cus, bool kept) {
    const Launch full = whole_launch(M, N, false, 256, 256);
    if (full.kind == kRefused) return full;
    double least = 0, time = 0;
    const bool small = small_layer(N, K);
    const LaunchTime& short_time = small ? kShortDownSmallTime : kept ? kShortDownKeptTime :
                                   M < long_from(N, K) ? kShortDownTime : kShortDownLongTime;
    const int form = choose_short_form(M, N, K, false, short_time, cus, least, small ? kSmallDownForms : 0);
    const double short_least = least;
    if (&short_time == &kShortDownTime) least *= kOverWhole;
    // The width: by time where the widest take no more than one round; over several rounds by rounds x columns, a column of
    // a narrower tile charged what it was measured to cost more for the token fragments it shares among fewer MFMAs
    // (12400 rows x 4096 columns: 3.6 rounds of 224-wide tiles 1033 us, 5 of 160-wide ones 1113 us).
    // Rectangular tiles by their time, from the fewest rows of the fit on; not for layers that stay in the Infinity Cache, whose
    // launches end before a large tile's rings have filled (1000 rows x 256 columns, K = 1024: 10.4 us, short 6.3).
    constexpr int per_mille[5] = {1000, 1020, 1070, 1170, 1310};
    const int rects = M < 1000 || small ? 0 : rect_forms(false);
    int width = 0;
    int64_t columns = 0;
    ShortShape rect = {0, 0, 1, 0};
    double rect_time = 0;
    for (int i = 0; i < 5 + rects; ++i) {
        const int w = 256 - 32 * i;
        const ShortShape f = i < 5 ? ShortShape{256, w, 1, 0} : rect_shape(false, i - 5);
        const TileGrid g = tile_grid(M, N, false, f);
        const double t = launch_time(g, M, K, false, f, i < 5 ? kFullDownTime : kRectDownTime, cus);
        if (t < 0) continue;
        if (i >= 5) {
            const double r = t * kRectDownPerMille[i - 5] / 1000;
            if (rect.tm == 0 || r < rect_time) { rect = f; rect_time = r; }
            continue;
        }
        const int64_t c = rounds_per_mille((int64_t)g.tiles, cus) * w * per_mille[i];
        if (width == 0 || (full.grid.tiles > (uint64_t)cus ? c < columns : t < time)) { width = w; time = t; columns = c; }
    }
    if (rect.tm && rect_time < kOverDown * time && (form < 0 || rect_time < kOverDown * least)) return timed(whole_launch(M, N, false, rect.tm, rect.tn), rect_time);
    if (form >= 0 && least < time) return timed(short_launch(M, N, false, form), short_least);
    return timed(whole_launch(M, N, false, 256, width), time);
}

// Gate/up with 256-row tiles: the first columns in tiles of 128 columns, the rest in tiles of 96, in one launch of
// the two-width kernel, where the same model says that saves time: 14336 columns with 12 token tiles are 1344 tiles
// = 5.25 rounds, but 64 x 128 + 64 x 96 columns are three rounds of each width.
// Few token rows: the short forms, as for the down projection.  Or 128 x 128 tiles, two workgroups per CU, by the same
// comparison.  more: the call has more than one mini-sequence.
inline Launch choose_gateup(int64_t M, int64_t N, int64_t K, int cus, bool more) {
    const Launch plain_launch = whole_launch(M, N, true, 256, 256);
    if (plain_launch.kind == kRefused) return plain_launch;
    double least = 0;
    const bool small = small_layer(N, K), one_group = to_pass_by(M, N, K, more);
    const int form = choose_short_form(M, N, K, true, small ? kShortGateUpSmallTime : kShortGateUpTime, cus, least, 0, one_group);
    const int64_t tm = plain_launch.grid.tiles_m;
    const double plain_time = launch_time(plain_launch.grid, M, K, true, {256, 256, 1, 0}, kFullGateUpTime, cus);
    // (no mix takes less than half of what the plain tiles take: where the short form does, it is not looked for)
    const bool few = form >= 0 && least < 0.5 * plain_time;
    const int64_t plain = rounds_per_mille(tm * ((N + 127) / 128), cus) * 128 * 1000;
    int64_t cost = plain;
    const int64_t narrow_tiles_n = few ? 0 : narrow_tiles(N, tm, cus, cost);
    const int64_t rest = N - 96 * narrow_tiles_n, wide_cols = rest > 0 ? (rest + 127) / 128 * 128 : 0;
    double full = plain_time * cost / plain;
    if (wide_cols == 0)
        full = launch_time(tile_grid(M, N, true, {256, 192, 1, 0}), M, K, true, {256, 192, 1, 0}, kFullGateUpTime, cus);
    // Rectangular tiles, by their time, for layers that come from HBM: 300 rows x 14336 columns, K = 4096: 91 -> 67 us; of a
    // layer of 69 MiB, which the Infinity Cache keeps, 1 % at most and up to 17 % lost at 128 rows.  Below 97 rows only where they keep the CUs busy.
    if (M >= 24 && 6 * N * K > ((int64_t)128 << 20)) {
        double rect = 0;
        const ShortShape r = choose_rect_form(M, N, K, true, kRectGateUpTime, cus, rect, one_group);
        const uint64_t tiles = r.tm ? tile_grid(M, N, true, r).tiles : 0;
        const bool filled = M <= 128 && tiles <= (uint64_t)cus && 8 * tiles >= 7 * (uint64_t)cus;
        if (filled && rect < kRectBytes * N * K) rect = kRectBytes * N * K;
        const double share = plain_launch.grid.tiles > (uint64_t)cus ? kOverOneRound : M <= 256 ? kOneTokenTile : kWithinOneRound;
        if (r.tm && (M > 96 || filled) && rect < share * full && (form < 0 || least >= full || rect < (filled ? kOverShortFilled : kOverShort) * least))
            return timed(whole_launch(M, N, true, r.tm, r.tn), rect);
    }
    const Launch pair = whole_launch(M, N, true, 128, 128);
    if (pair.kind != kRefused && !(one_group && pair.grid.tiles_m > (uint32_t)kTokenGroup) && pair.grid.tiles <= 2 * (uint64_t)cus &&
        (K <= 2048 || (pair.grid.tiles_m > (uint32_t)kTokenGroup && pair.grid.tiles > (uint64_t)cus))) {
        const double t = launch_time(pair.grid, M, K, true, kPairShape, small ? kPairGateUpSmallTime : kPairGateUpTime, cus);
        if (t < full && (form < 0 || t < least)) return timed(pair, t);
    }
    if (form >= 0 && least < full) return timed(short_launch(M, N, true, form), least);
    if (narrow_tiles_n == 0 || wide_cols >= N) return timed(plain_launch, plain_time);
    if (wide_cols == 0) return timed(whole_launch(M, N, true, 256, 192), full);
    Launch l = {kTwoWidths, 0, 256, 256, wide_cols, tile_grid(M, wide_cols, true, {256, 256, 1, 0}),
                tile_grid(M, N - wide_cols, true, {256, 192, 1, 0}), full};
    if (l.grid.tiles > (uint64_t)kMaxTiles || l.narrow.tiles > (uint64_t)kMaxTiles) l.kind = kRefused;
    return l;
}

// ---- Passes of more rows than the workspace holds: `out` behind the rows of a pass is not computed yet, and the rest of its
// intermediate can lie there.
//
// A pass of R of the `left` rows that are still to do puts its rows from `split` on at the end of `out`, which must not reach down to row R:
// 2 (R - split) I bytes, and up to 256 for the alignment, of the 2 (left - R) H that are free.  A longer pass takes less time per row, down to
// some 4096 of them: one mini-sequence at a time -> so, H = 4096, I = 14336: 8192 rows by 128 5635 us -> 2970, by 512 2552 -> 2335, 32768 by
// 512 10215 -> 8062, 16384 by 1024 4364 -> 4090, with the workspace of two 4136 -> 4009; H = 1056, I = 2080: 8192 by 512 351 -> 193.
constexpr int64_t kSpareAlign = 256;
inline int64_t most_rows(int64_t left, int64_t H, int64_t I, int64_t split) { return (left * H + split * I - kSpareAlign / 2) / (H + I); }

constexpr int64_t kWhole = 0x7fffffff;
struct Pass {
    int64_t rows = 0, split = 0;         // rows 0: none; split kWhole: all rows lie in the workspace
    Launch gateup, down;
    double time() const { return gateup.time + down.time; }
};
// Rows of the pass that lie in the workspace of C rows: whole token tiles of the down launch, so that none of them needs both pieces.
inline int64_t split_of(const Launch& down, int64_t C) { return C / down.tm * down.tm; }

// Whether to ask for longer passes at all (1 ... 4 us on the host for each one looked at): where there is one, of calls of some 20 us and
// more, and with mini-sequences of less than about 0.9 ms, which a longer pass betters by a percent at most (H = 4096, I = 14336: 3000 rows
// 0 ... 2.4 %, 4096 none).
inline bool longer_passes(int64_t S, int64_t H, int64_t I, int64_t C) {
    return S > C && S * H >= ((int64_t)1 << 31) / I && C * H < ((int64_t)3 << 36) / I && most_rows(S, H, I, C / 256 * 256) / 256 * 256 > C;
}

// The passes of a call of S rows with a workspace for C of them, one after the other: what the driver runs, and what is weighed against
// blocks.  Passes of C rows (or what is left), and longer ones, if `longer` and longer_passes say so.
class Passes {
public:
    int64_t left;                        // rows still to do

    Passes(int64_t S, int64_t H, int64_t I, int64_t C, int cus, bool longer)
        : left(S), H(H), I(I), C(C), cus(cus), more_(S > C), longer_(longer && longer_passes(S, H, I, C)) {
        gateup_ = choose_gateup(C, I, H, cus, more_);
        down_ = choose_down(C, H, I, cus, false);
        kept_ = S > kKeptFrom * C && !small_layer(I, H) && kept_down(gateup_, C, H, I) ? choose_down(C, H, I, cus, true) : down_;
    }
    // The next pass, and (plain) what it is where no longer one is looked for.
    Pass next() {
        const Pass p = has_room() ? longer_pass() : Pass();
        if (!p.rows) return plain();
        // Where the first saves no two passes, longer ones are weighed against none; where they save too little, none are looked for again.
        if (!taken_ && p.rows < 2 * C && !they_save_time(p)) {
            longer_ = false;
            return plain();
        }
        return p;
    }
    Pass plain() const { return of_rows(left < C ? left : C, since_); }
    // Go on behind p (next or plain, its launches may be others of the same rows).
    void done(const Pass& p) {
        left -= p.rows;
        taken_ |= p.split != kWhole;
        since_ = p.split == kWhole || kept_down(p.gateup, p.rows, H, I) ? since_ + 1 : 0;
    }
    // What all that is left is expected to take, us, if that is less than `limit`.  Whether it is is known as soon as the rest would be so
    // without longer passes (and this is returned), or, since shorter passes take more time per row, reaches the limit at 0.9 of the last
    // one's: mostly behind the first.  All take 20 ... 100 us on the host.
    double time(double limit = kAll) const {
        Passes then = *this;
        double t = 0;
        while (then.has_room()) {
            const Pass p = then.next();
            t += p.time();
            then.done(p);
            if (t + 0.9 * p.time() / p.rows * then.left >= limit) return limit;
            if (limit < kAll && t + then.plain_time(then.left, then.since_) < limit) break;
        }
        return t + then.plain_time(then.left, then.since_);
    }
    static constexpr double kAll = 1e30;

private:
    Pass of_rows(int64_t rows, int64_t since) const {
        Pass p;
        p.rows = rows;
        p.split = kWhole;
        if (rows == C) {
            p.gateup = gateup_;
            p.down = since >= kKeptFrom ? kept_ : down_;
        } else {
            p.gateup = choose_gateup(rows, I, H, cus, more_);
            p.down = choose_down(rows, H, I, cus, since >= kKeptFrom && kept_down(p.gateup, rows, H, I));
        }
        return p;
    }
    // `rows` of them without longer passes, behind `since` that kept W_down.
    double plain_time(int64_t rows, int64_t since) const {
        const int64_t n = rows / C, cold = since >= kKeptFrom ? 0 : n < kKeptFrom - since ? n : kKeptFrom - since, rest = rows % C;
        return cold * (gateup_.time + down_.time) + (n - cold) * (gateup_.time + kept_.time) + (rest ? of_rows(rest, since + n).time() : 0);
    }
    bool has_room() const { return longer_ && longest() > C; }
    int64_t longest() const { return most_rows(left, H, I, C / 256 * 256) / 256 * 256; }
    Pass longer_pass() const;
    bool they_save_time(const Pass& first) const;

    int64_t H, I, C;
    int cus;
    bool more_, longer_, taken_ = false; // more: the call has more than one mini-sequence; taken: one of its passes was longer
    int64_t since_ = 0;                  // passes since the last that displaced W_down
    Launch gateup_, down_, kept_;        // of C rows; kept: with W_down in the Infinity Cache, where it stays there
};

// The pass of whole 256-row tiles, more than C rows, that takes the least time per row, of the three longest; none where
// it is not 3 % less than in the pass of C rows that would be the next.  Of 651 calls of eight layers 246 took less time so, 19 % on average, where
// that pass was taken to find W_down in the Infinity Cache, which the first ones don't (512 rows of H = 3584, I = 18944: 0.445 us a row and 0.385).  With
// what it takes itself 241 more of 1785 calls of eleven layers change, 193 of them by more than 1 %, to 3 % less time on average, and 7 by
// more than 1 % for the worse (2.2 % at most).
inline Pass Passes::longer_pass() const {
    Pass best;
    double least = 0.97 * of_rows(C, since_).time() / C;
    int64_t rows = longest();
    for (int i = 0; i < 3 && rows > C; ++i, rows -= 256) {
        Pass p;
        p.rows = rows;
        p.gateup = choose_gateup(rows, I, H, cus, true);
        p.down = choose_down(rows, H, I, cus, false);
        if (p.gateup.kind == kRefused || p.down.kind == kRefused) continue;
        p.split = split_of(p.down, C);
        const double t = p.time() / rows;
        if (t < least && rows <= most_rows(left, H, I, p.split)) { best = p; least = t; }
    }
    return best;
}

// Whether the whole call takes less time with longer passes, `first` the first of them.  They leave another last pass behind: 3072 rows
// of H = 512, I = 1536 by 1024 went as 1280 + 1024 + 768 in 46.6 us, as three of 1024 take 44.1, and 7471 by 2500 as 3584 + 2500 + 1387
// in 67.9, 62.0 as mini-sequences.  With as many passes they have to save 1 % of all, less than which the formula does not
// tell (its error is 5 ... 8 % of a launch); with fewer, anything, and a pass counts 5 us less than its launches by themselves, which is what they
// take less one behind the other in layers that the Infinity Cache holds (measured 4 ... 8).  Of 1785 calls of eleven layers 61 change: 23 had
// lost 1 ... 10 % by longer passes and have it back, but for 6 that still lose 1.0 ... 1.7 %; 15 had gained 1 ... 4.6 %, which go (2000 rows of H = 1056, I =
// 2080 by 800 66.4 -> 69.9 us).
inline bool Passes::they_save_time(const Pass& first) const {
    const double otherwise = plain_time(left, since_), overlap = 6 * H * I <= ((int64_t)256 << 20) ? 5 : 0;
    Passes then = *this;
    double t = 0;
    int64_t n = 0;
    for (Pass p = first; p.rows; p = then.has_room() ? then.longer_pass() : Pass()) {
        t += p.time();
        ++n;
        then.done(p);
        const int64_t fewer = (left + C - 1) / C - n - (then.left + C - 1) / C;
        const double saved = otherwise - t - then.plain_time(then.left, then.since_) - overlap * fewer;
        if (saved >= (fewer > 0 ? 0 : 0.01 * otherwise)) return true;
    }
    return false;
}

// ---- Whole blocks of token rows in one launch (mom_block.hip.inc), for calls of several mini-sequences on a small layer.
constexpr int kBlockPad = 8;            // elements behind an LDS row: 16 bytes, so that 16 rows at one k lie on different banks
constexpr int kBlockUnit = 4096;        // bytes of a unit of weights
// Bytes of LDS of a block of `rows` token rows and `units` units of weights.
constexpr int64_t block_lds(int64_t rows, int64_t H, int64_t I, int units) {
    return rows * (H + I + 2 * kBlockPad) * 2 + (int64_t)units * kBlockUnit;
}
// X(TB, WAVES, R): 16 TB token rows, WAVES wavefronts with rings of R units.  bytes_per_us: weights through a workgroup, measured at
// H = 256, I = 1024 (16 rows 18.3 us for 512 token rows, 32 rows 24 us for 8192) and H = 1056, I = 2080 (166 us for 3000 with the weights
// in the Infinity Cache, 240 where other layers have displaced them).  Tokens
// in and out take 1 us per 10^6 elements more.
#define MOM_BLOCK_FORMS(X) X(1, 8, 2) X(2, 8, 2) X(1, 6, 2)
struct BlockForm { int tb, waves, r, bytes_per_us; };
#define MOM_SHAPE(TB, WAVES, R) {TB, WAVES, R, TB == 2 ? 95000 : WAVES == 8 ? 110000 : 79000},
constexpr BlockForm kBlockForms[] = {MOM_BLOCK_FORMS(MOM_SHAPE)};
#undef MOM_SHAPE
constexpr int kBlockFormCount = sizeof(kBlockForms) / sizeof(kBlockForms[0]);
inline bool block_fits(const BlockForm& f, int64_t H, int64_t I) { return H + I <= 8192 && block_lds(16 * f.tb, H, I, f.waves * f.r) <= 163840; }
// (32-bit arithmetic, as in tile_grid: a call of one launch is not much longer than the choice.)
inline uint32_t block_count(const BlockForm& f, int64_t S) { return ((uint32_t)S + 16 * f.tb - 1) / (16 * (uint32_t)f.tb); }
// Groups of 32 output columns per workgroup: where CUs are left idle, up to eight workgroups share those of a block, four groups each at least (half
// the wavefronts have one then).  H = 256, I = 1024, 512 rows: one workgroup per block 18.3 us, two 16.8, four 16.9, eight 17.4; H = 1056, I = 2080:
// one 174, two 142, four 129, eight 124; 1024 rows in four 133 instead of 169.
inline int block_share(uint32_t blocks, int64_t H, int cus) {
    const uint32_t groups = (uint32_t)H / 32;
    if (groups <= 4 || 2 * blocks > (uint32_t)cus) return (int)groups;
    const uint32_t spare = (uint32_t)cus / blocks, parts = spare > 8 ? 8 : spare, share = (groups + parts - 1) / parts;
    return (int)(share > 4 ? share : 4);
}
inline uint32_t block_parts(int64_t H, int share) { return ((uint32_t)H / 32 + share - 1) / (uint32_t)share; }
// With shares a microsecond per 16 rows goes to the shorter last phase (H = 256, I = 1024, 32 rows: 19.8 us in two, 18.8 without it).
inline double block_time(const BlockForm& f, int64_t S, int64_t H, int64_t I, int cus) {
    const uint32_t blocks = block_count(f, S);
    const int share = block_share(blocks, H, cus);
    const double bytes = 4.0 * H * I + 64.0 * I * share;
    return 4.0 + (double)((blocks + cus - 1) / (uint32_t)cus) * bytes / f.bytes_per_us + 1.0e-6 * S * H + (share < H / 32 ? f.tb : 0);
}

// The form in which S token rows take less time than as mini-sequences of C of them, whose two launches are given; -1: none.  longer: or as longer passes.  A
// mini-sequence takes 6 us less than the launches by themselves (H = 256, I = 1024: 128 rows 7.0 us, 512 8.0, 2048 11.0, formula
// 13.1, 14.2, 17.2; H = 1056, I = 2080: 128 rows 12.3, formula 18.1; where both are longer, 512 rows 21.5 and 24.7, the loop
// looks better than it is).  7 % off that: 2048 rows by 1024 of the former 17.2 us, formula 18.9, as blocks 18.7.  Up to 24576 rows
// by mini-sequence: 40000 rows by 18022 take 104 us in blocks, 118 as mini-sequences, but 66000 by 26214 185 and 178, 34000 by 32440 102
// and 92, which the formula overrates.
constexpr int64_t kBlockLongest = 24576;
inline int choose_block(int64_t S, int64_t H, int64_t I, int64_t C, int cus, const Launch& gateup, const Launch& down, bool longer = true) {
    if (S <= C || C > kBlockLongest || !small_layer(I, H)) return -1;
    int best = -1;
    double least = 0;
    for (int i = 0; i < kBlockFormCount; ++i) {
        const BlockForm& f = kBlockForms[i];
        if (!block_fits(f, H, I) || (int64_t)block_count(f, S) * f.waves * 64 > (int64_t)0x7fffffff) continue;
        const double t = block_time(f, S, H, I, cus);
        if (best < 0 || t < least) { best = i; least = t; }
    }
    if (best < 0) return -1;
    const double one = gateup.time + down.time - 6;
    if (least >= 0.93 * one * ((S + C - 1) / C)) return -1;
    // Longer passes, asked for only where the blocks take several rounds of the CUs: 8192 rows of H = 1056, I = 2080 by 256 339 us in
    // blocks, 224 so, 16384 673 and 335.
    if (longer && block_count(kBlockForms[best], S) > (uint32_t)cus && longer_passes(S, H, I, C) && Passes(S, H, I, C, cus, true).time(least) < least) return -1;
    return best;
}

// ---- Token rows of a pass of mom_mlp_prefill_static and mom_mlp_prefill_pipelined, whose workspaces hold more than mini_seq of them.

// What a call of S rows, R at a time, is expected to take, us, if that is less than `limit`.  longer: by the passes that run, or without longer
// ones.
inline double call_time(int64_t S, int64_t H, int64_t I, int64_t R, int cus, bool longer, double limit = Passes::kAll) {
    const Passes passes(S, H, I, R, cus, longer);
    if (S > R && small_layer(I, H)) {
        const Pass p = passes.plain();
        const int form = choose_block(S, H, I, R, cus, p.gateup, p.down, longer);
        if (form >= 0) return block_time(kBlockForms[form], S, H, I, cus);
    }
    return passes.time(limit);
}

// `rows` at a time, or, of as few passes as a workspace for `most` rows allows, all of the same length in whole 256-row tiles, where that is
// expected to take 3.5 % less.  1350 rows of H = 6144, I = 16384 by 600 take 857 us, as 512, 512 and 326 695; static, 33875 rows of H =
// 1056, I = 2080 by 16128 416, by 11520 379.  Of 1557 calls with two mini-sequences' workspace (S 1.05 ... 4.5 C, 14 layers) 165 change, by
// 5.5 % on average, 4 for the worse by 2 % or a little more; with 1 % promised 319, 17 for the worse.  That is without longer passes; where
// there may be some, not if these take less time with `rows`, whose workspace holds more: 7757 rows of H = 2048, I = 8192 by 2578, as 3072, 2816 and
// 1869 of them, 572 us, by 2048 602.  Of 1633 calls of twelve layers 26 take `rows` so, none in more time (3 % less).  Of more than 64 passes
// that is not asked, as each may have to be looked at.  Nothing is asked of calls of less than some 40 us, which the asking (3 ... 10 us on the
// host, 20 ... 60 with longer passes) would make longer: 690 rows of a 256 x 1024 layer 16.1 -> 17.5 us.
inline int64_t even_rows(int64_t S, int64_t H, int64_t I, int64_t rows, int64_t most, int cus) {
    const int64_t n = (S + most - 1) / most, even = ((S + n - 1) / n + 255) / 256 * 256;
    if (n == 1 || even >= most || even == rows || S * H < ((int64_t)1 << 33) / I) return rows;
    if (call_time(S, H, I, even, cus, false) >= 0.965 * call_time(S, H, I, rows, cus, false)) return rows;
    if (rows < even || n > 64 || !longer_passes(S, H, I, rows)) return even;
    const double t = call_time(S, H, I, even, cus, true);
    return call_time(S, H, I, rows, cus, true, t) < t ? rows : even;
}

// Static: the array of `bytes` is there at its full size whatever mini_seq (C rows) is, and a pass of more rows takes less time per row
// (H = 4096, I = 14336, 12000 rows: by 128 rows 8054 us, by 512 3832, by 1024 3202, by 2304 2970).  Whole 256-row token tiles, and only from
// half as many rows again on: at 8192 -> 16128 rows of I = 2080 14 % are gained.
inline int64_t static_rows(int64_t S, int64_t H, int64_t I, int64_t C, int64_t bytes, int cus) {
    const int64_t fit = bytes / (2 * I), whole = fit / 256 * 256;
    if (S <= fit) return S;
    return whole ? even_rows(S, H, I, 2 * whole >= 3 * C ? whole : C, whole, cus) : C;
}

// Two mini-sequences' workspace: both at once, up to 14 rounds of the CUs in 256 x 128 gate/up tiles of one of them.  Against the
// workspace as a double buffer, down(c) beside gate/up(c+1) on two streams, H = 4096, I = 14336, six mini-sequences of C rows: C = 512 979 -> 824 us, 1024 1675 ->
// 1545, 2048 3043 -> 2734, 4096 level; H = 3584, I = 18944: 512 1261 -> 1020, 2048 3609 -> 3244, 6000 10109 -> 9676.  From 14 rounds on a
// pass more costs less than 1 %, and 18000 rows at once 3 % more than 12000 and 6000.
inline int64_t pipelined_rows(int64_t S, int64_t H, int64_t I, int64_t C, int cus) {
    if (S <= C) return S;
    const int64_t tiles = (int64_t)whole_launch(C, I, true, 256, 256).grid.tiles, both = 2 * C < S ? 2 * C : S;
    return even_rows(S, H, I, tiles >= 14 * (int64_t)cus ? C : both, both, cus);
}

}  // namespace momk

#endif  // MOM_GEMM_FORMS_H

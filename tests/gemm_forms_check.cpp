// Host check of the short GEMM forms and of the rule that picks one (csrc/mom_gemm_forms.h): what a form assumes
// about its sizes, and that every launch size gets a form that the kernels can run.
#include <cstdio>
#include <cmath>
#include <initializer_list>
#include <vector>
#include "mom_gemm_forms.h"

static int bad = 0;
#define CHECK(c, ...) do { if (!(c)) { printf("FAILED %s: ", #c); printf(__VA_ARGS__); printf("\n"); ++bad; } } while (0)

// The requests of a ring in the order of the kernel: every load of a stage once, into a slot whose stage is in registers, and each wait is for
// the stage that is needed next and no other.
static void ring(int tm, int tn, int nstg, int loads, int group) {
    std::vector<int> stage;                           // of every load, in the order of the requests
    auto request = [&](int first, int n) {
        for (int j = 0; j < loads; ++j)
            for (int g = 0; g < n; ++g) stage.push_back(first + g);
    };
    auto landed = [&](int t, int in_flight) {         // loads up to all of stage t, and how many are not waited for
        int behind = 0;
        for (size_t i = stage.size(); i > 0 && stage[i - 1] != t; --i) ++behind;
        CHECK(in_flight == (behind > 63 ? 63 : behind), "%d x %d, %d stages, groups of %d: stage %d waited for at %d in flight, %d behind it", tm, tn, nstg,
              group, t, in_flight, behind);
    };
    for (int t = 0; t < nstg; ++t)
        if (t == 0 || momk::ring_place(t, nstg, group) == 0) request(t, group - momk::ring_place(t, nstg, group));
    landed(0, momk::ring_in_flight(0, nstg - 1, nstg, group, loads));
    for (int t = 0; t < 40; ++t) {
        // (the phases of the kernel: t % group stands for t)
        landed(t + 1, momk::ring_in_flight(t % group + 1, momk::ring_ahead(t % group, nstg, group), nstg, group, loads));
        const int first = momk::ring_first(t, nstg, group);
        const int phase = t % group, phase_first = momk::ring_first(phase, nstg, group);
        CHECK((first < 0) == (phase_first < 0) && (first < 0 || phase_first - phase == first - t), "requests at stage %d and at its phase", t);
        if (first < 0) continue;
        for (int g = 0; g < group; ++g)               // slot of stage first + g: that of stage first + g - nstg, in the kernel's count t - group + 1 + g
            CHECK(first + g - nstg == t - group + 1 + g && first + g - nstg <= t, "slot of stage %d at stage %d, %d stages", first + g, t, nstg);
        request(first, group);
    }
    std::vector<int> seen(stage.back() + 1);
    for (int t : stage) ++seen[t];
    for (size_t t = 0; t < seen.size(); ++t) CHECK(seen[t] == loads, "stage %d of %d x %d requested %d times", (int)t, tm, tn, seen[t] / loads);
}

static void form(bool gu, int f, int tm, int tn, int wm, int wn, int ksub, int nstg) {
    const int stage = ksub * (tm + tn) * 128, loads = ksub * (tm + tn) / 32;
    const int cols = gu ? tn / 2 : tn;
    CHECK(nstg * stage <= 163840 && stage <= 65536 && nstg >= 2, "ring of %d x %d", tm, tn);
    CHECK((nstg - 2) * loads <= 63, "loads in flight of %d x %d", tm, tn);
    for (int group : {1, 2})
        if (group == 1 || (gu && nstg >= 5)) ring(tm, tn, nstg, loads, group);
    CHECK(wm * wn <= 4 && tm % (16 * wm) == 0 && tn % (16 * wn) == 0, "wavefront grid of %d x %d", tm, tn);
    CHECK(!gu || (tn / 16 / wn) % 2 == 0, "gate and up blocks of %d x %d", tm, tn);
    CHECK((ksub * tm) % 32 == 0 && (ksub * tn) % (gu ? 64 : 32) == 0, "loads per wavefront of %d x %d", tm, tn);
    CHECK(tm * (cols * 2 + 16) <= nstg * stage, "epilogue of %d x %d", tm, tn);
    const momk::ShortShape s = momk::short_shape(gu, f);
    CHECK(s.tm == tm && s.tn == tn && s.per_cu >= 1 && s.per_cu * nstg * stage <= 163840, "workgroups per CU of %d x %d", tm, tn);
    // Every 1-KiB block of a stage is loaded once, to a place of its own, from the row that belongs there
    bool seen[2][16][64] = {};                        // [operand][sub][row / 8]
    int moved = 0;
    for (int wave = 0; wave < 4; ++wave)
        for (int j = 0; j < loads; ++j, ++moved) {
            const momk::RingLoad l = momk::ring_load(gu, tm, tn, ksub, wave, j);
            const bool up = gu && !l.token && momk::ring_load_up(tm, tn, ksub, j);     // from W_up
            CHECK(l.token == (j < ksub * tm / 32), "operand of a load of %d x %d", tm, tn);
            CHECK(l.sub >= 0 && l.sub < ksub && l.row >= 0 && l.row % 8 == 0 && l.row + 8 <= (l.token ? tm : tn), "block of %d x %d", tm, tn);
            CHECK(l.src == l.row - (up ? tn / 2 : 0) && (l.token || (l.src >= 0 && l.src + 8 <= cols)), "source of a load of %d x %d", tm, tn);
            CHECK(!seen[l.token][l.sub][l.row / 8], "block loaded twice in %d x %d", tm, tn);
            seen[l.token][l.sub][l.row / 8] = true;
        }
    CHECK(moved * 8 == ksub * (tm + tn), "blocks of %d x %d", tm, tn);
}

// The workgroups of a launch run every tile of the grid once, and the token tiles cover every token row once: tile i
// starts at row i tm.
static void tiles(int64_t M, int64_t N, int tm, int tn) {
    const momk::TileGrid g = momk::tile_grid(M, N, false, {tm, tn, 1, 0});
    CHECK(g.tiles == (uint64_t)g.tiles_m * g.tiles_n, "tiles of M=%lld tm=%d", (long long)M, tm);
    const int xcd = momk::tiles_per_xcd(g.tiles), count = (int)g.tiles;
    std::vector<int> run(count);
    std::vector<char> token(M), column(N);
    for (int bid = 0; bid < 8 * xcd; ++bid) {
        const int vt = momk::tile_number(bid, xcd);
        if (vt >= count) continue;
        const momk::TilePlace p = momk::tile_place(vt, g.tiles_m, g.tiles_n, momk::kTokenGroup);
        const bool in = p.m >= 0 && p.n >= 0 && p.m < (int)g.tiles_m && p.n < (int)g.tiles_n;
        CHECK(in, "place of tile %d of M=%lld tm=%d", vt, (long long)M, tm);
        if (!in) return;
        CHECK(!run[p.m * g.tiles_n + p.n]++, "tile %d x %d of M=%lld tm=%d run twice", p.m, p.n, (long long)M, tm);
        CHECK((int64_t)p.m * tm < M && (int64_t)p.n * tn < N, "empty tile %d x %d of M=%lld tm=%d", p.m, p.n, (long long)M, tm);
        for (int64_t m = (int64_t)p.m * tm; m < M && m < (int64_t)(p.m + 1) * tm; ++m) token[m] = 1;
        for (int64_t n = (int64_t)p.n * tn; n < N && n < (int64_t)(p.n + 1) * tn; ++n) column[n] = 1;
    }
    int64_t ran = 0, rows = 0, cols = 0;
    for (int r : run) ran += r;
    for (char c : token) rows += c;
    for (char c : column) cols += c;
    CHECK(ran == count, "tiles run of M=%lld tm=%d", (long long)M, tm);
    CHECK(rows == M && cols == N, "rows of M=%lld tm=%d", (long long)M, tm);
}

// What choose_down picks at these sizes, against every launch there is, each priced on the grid that runs.
static int64_t rounds(const momk::TileGrid& g, int cus) { return ((int64_t)g.tiles + cus - 1) / cus; }
static void down_choice(int64_t M, int64_t N, int64_t K, int cus, bool more) {
    const momk::Launch l = momk::choose_down(M, N, K, cus, more && momk::kept_down(momk::choose_gateup(M, K, N, cus, true), M, N, K));
    CHECK(l.kind == momk::kShortTiles || l.kind == momk::kWholeTiles, "down M=%lld N=%lld", (long long)M, (long long)N);
    if (l.kind == momk::kWholeTiles) return;
    // With a long contraction a 256-row tile takes at most a little more than a short one of the same width, so short
    // tiles that need more rounds than 256-row tiles no wider than 192 are never the faster ones (measured at 2400 ... 5500 rows).
    for (int w : {192, 160, 128})
        CHECK(l.tm * l.tn < 160 * 128 || rounds(l.grid, cus) <= rounds(momk::tile_grid(M, N, false, {256, w, 1, 0}), cus),
              "down M=%lld N=%lld K=%lld: %d x %d in %lld rounds, 256 x %d in %lld", (long long)M, (long long)N, (long long)K, l.tm, l.tn,
              (long long)rounds(l.grid, cus), w, (long long)rounds(momk::tile_grid(M, N, false, {256, w, 1, 0}), cus));
}

// Neighbouring row counts don't alternate between two launches.
static void steady(int64_t N, int64_t K, bool gateup) {
    momk::Launch before = {}, last = {};
    int64_t since = 0;
    auto same = [](const momk::Launch& a, const momk::Launch& b) {
        return a.kind == b.kind && a.form == b.form && a.tm == b.tm && a.tn == b.tn && a.wide_cols == b.wide_cols;
    };
    for (int64_t M = 1; M <= 8192; ++M) {
        const momk::Launch l = gateup ? momk::choose_gateup(M, N, K, 256, false) : momk::choose_down(M, N, K, 256, false);
        if (M > 1 && same(l, last)) continue;
        CHECK(!since || !same(l, before) || M - since >= 4, "M=%lld N=%lld K=%lld: %d x %d between two runs of %d x %d", (long long)since,
              (long long)N, (long long)K, last.tm, last.tn, l.tm, l.tn);
        before = last;
        last = l;
        since = M;
    }
}

// W_down is taken to be in the cache behind launches that pass it by only, and mini-sequences of one group of token tiles pass it by.
static void kept(int64_t H, int64_t I) {
    for (int64_t M = 1; M <= 3000; ++M) {
        const momk::Launch l = momk::choose_gateup(M, I, H, 256, true);
        const bool once = momk::weights_once(l.grid.tiles_m, I, H, true), down = momk::kept_down(l, M, H, I);
        if (6 * H * I <= (256 << 20)) continue;
        CHECK(!down || once, "W_down kept M=%lld H=%lld I=%lld: gate/up %d x %d", (long long)M, (long long)H, (long long)I, l.tm, l.tn);
        CHECK(!momk::to_pass_by(M, I, H, true) || down, "W_down displaced M=%lld H=%lld I=%lld: gate/up %d x %d", (long long)M, (long long)H,
              (long long)I, l.tm, l.tn);
    }
}

// The mix of tiles of 128 and 96 columns that narrow_tiles finds by counting on, and its cost, against every mix by itself.
static void mixes(int64_t N, int64_t tm, int cus) {
    auto mix_cost = [&](int64_t b) {
        const int64_t rest = N - 96 * b, wide = rest > 0 ? (rest + 127) / 128 : 0;
        return momk::rounds_per_mille(tm * wide, cus) * 128 * 1000 + momk::rounds_per_mille(tm * b, cus) * 96 * momk::kGateUpNarrowPerMille;
    };
    int64_t cost = mix_cost(0), best = 0, got = 0;
    for (int64_t b = 1; b <= (N + 95) / 96; ++b)
        if (mix_cost(b) < cost && mix_cost(b) * 1000 <= mix_cost(0) * (1000 - momk::kGateUpMixMinGainPerMille)) { cost = mix_cost(b); best = b; }
    const int64_t b = momk::narrow_tiles(N, tm, cus, got);
    CHECK(b == best && got == cost, "N=%lld in %lld token tiles on %d CUs: %lld narrow tiles, not %lld", (long long)N, (long long)tm, cus, (long long)b, (long long)best);
}

// Rows of a pass fit the workspace, and what was measured the faster of the candidates is taken.
static void passes() {
    const int64_t layers[][2] = {{4096, 14336}, {3584, 18944}, {6144, 16384}, {3584, 9728}, {1056, 2080}, {256, 1024}, {32, 1 << 20}, {1 << 20, 32}};
    int even = 0, more = 0;
    for (const auto& l : layers)
        for (int64_t C = 1; C < 40000; C += 1 + C * 3 / 7)
            for (int64_t S : {C + 1, 2 * C - 1, 2 * C, 2 * C + 1, 3 * C + C / 3, 9 * C, 100 * C + 7, (int64_t)0x7fffff00}) {
                if (S <= C) continue;
                const int64_t p = momk::pipelined_rows(S, l[0], l[1], C, 256), bytes = 64 << 20;
                CHECK(p >= 1 && p <= 2 * C && p <= S, "pipelined S=%lld C=%lld: %lld rows", (long long)S, (long long)C, (long long)p);
                even += p != C && p != 2 * C && p != S;
                if (2 * C * l[1] > bytes) continue;
                const int64_t t = momk::static_rows(S, l[0], l[1], C, bytes, 256);
                CHECK(t >= 1 && t <= S && 2 * t * l[1] <= bytes, "static S=%lld C=%lld I=%lld: %lld rows", (long long)S, (long long)C, (long long)l[1], (long long)t);
                more += t > C;
            }
    CHECK(even > 50 && more > 100, "%d even, %d larger", even, more);
    const int64_t two[][5] = {{1350, 6144, 16384, 300, 512}, {1350, 4096, 14336, 300, 512}, {4050, 8192, 28672, 1500, 2048}, {8100, 4096, 14336, 3000, 4096},
                              {3072, 4096, 14336, 512, 1024}, {16384, 4096, 14336, 1024, 2048}, {32768, 4096, 14336, 8192, 8192}};
    for (const auto& t : two) {
        const int64_t r = momk::pipelined_rows(t[0], t[1], t[2], t[3], 256);
        CHECK(r == t[4], "pipelined S=%lld C=%lld: %lld rows, not %lld", (long long)t[0], (long long)t[3], (long long)r, (long long)t[4]);
    }
    // Passes of the same length give way where the driver's longer passes take less time with all of the workspace.
    const int64_t whole[][5] = {{18497, 1056, 2080, 4391, 8782}, {7757, 2048, 8192, 1289, 2578}, {15154, 512, 1536, 2143, 4286}, {3093, 1024, 4096, 772, 1544}};
    for (const auto& t : whole) {
        const int64_t r = momk::pipelined_rows(t[0], t[1], t[2], t[3], 256);
        CHECK(r == t[4], "pipelined S=%lld C=%lld: %lld rows, not %lld", (long long)t[0], (long long)t[3], (long long)r, (long long)t[4]);
    }
    for (const auto& l : layers)
        for (int64_t C = 100; C < 6000; C += 1 + C / 11)
            for (int64_t S = 2 * C + 1; S < 9 * C; S += 1 + C * 3 / 5) {
                const int64_t p = momk::pipelined_rows(S, l[0], l[1], C, 256);
                if (p == C || p == 2 * C || p == S) continue;
                const double even = momk::call_time(S, l[0], l[1], p, 256, true), both = momk::call_time(S, l[0], l[1], 2 * C < S ? 2 * C : S, 256, true);
                const double one = momk::call_time(S, l[0], l[1], C, 256, true);         // (long mini-sequences go one at a time)
                CHECK(even <= 1.0001 * both || even <= 1.0001 * one, "pipelined S=%lld C=%lld H=%lld: %lld rows %.1f us, %.1f with all", (long long)S, (long long)C,
                      (long long)l[0], (long long)p, even, both);
            }
    const int64_t fixed[][5] = {{33875, 1056, 2080, 128, 11520}, {20766, 1056, 2080, 10752, 10496}, {33875, 1056, 2080, 8000, 11520}, {12000, 4096, 14336, 128, 2304},
                                {2304, 4096, 14336, 128, 2304}, {2457, 4096, 14336, 128, 2304}, {12000, 4096, 14336, 2000, 2000}};
    for (const auto& t : fixed) {
        const int64_t r = momk::static_rows(t[0], t[1], t[2], t[3], 64 << 20, 256);
        CHECK(r == t[4], "static S=%lld C=%lld: %lld rows, not %lld", (long long)t[0], (long long)t[3], (long long)r, (long long)t[4]);
    }
}

int main() {
    for (int tm = 16; tm <= 256; tm += 16)
        for (int64_t M = 1; M <= 16384; M += 1 + M / 97) tiles(M, 96 + 32 * (M % 11), tm, 64);
    const momk::TileGrid most = momk::tile_grid(0x7fffff00, 32, false, {256, 32, 1, 0});
    CHECK(most.tiles_m == 0x7fffff && most.tiles_n == 1 && most.tiles == 0x7fffff, "most token rows");
    for (int64_t M = 1; M <= 16384; ++M) {
        for (bool more : {false, true}) down_choice(M, 4096, 14336, 256, more);
        for (bool more : {false, true}) down_choice(M, 3584, 18944, 256, more);
        for (bool more : {false, true}) down_choice(M, 8192, 28672, 256, more);
        CHECK(momk::choose_gateup(M, 14336, 4096, 256, false).kind != momk::kRefused, "gate/up M=%lld", (long long)M);
    }
    const int64_t layers[][2] = {{4096, 14336}, {3584, 18944}, {1056, 2080}, {256, 1024}};
    for (const auto& l : layers) {
        steady(l[0], l[1], false);
        steady(l[1], l[0], true);
    }
    const int64_t kept_layers[][2] = {{4096, 14336}, {3584, 18944}, {4096, 11008}, {6144, 16384}, {5120, 13824}, {5120, 25600}, {2048, 8192}};
    for (const auto& l : kept_layers) kept(l[0], l[1]);
    passes();
    for (int cus : {1, 80, 256, 304})
        for (int64_t N : {32, 96, 128, 160, 1024, 2080, 9728, 14336, 18944, 28672, 1 << 20})
            for (int64_t tm = 1; tm < (N > 30000 ? 600 : 8388608); tm += 1 + tm / 9) mixes(N, tm, cus);
    // Where the constants of the short down forms change, and from where the rectangular ones are looked at, the choice doesn't.
    const int64_t edge_layers[][2] = {{4096, 14336}, {3584, 18944}, {3584, 9728}, {2560, 9728}, {6144, 16384}, {4096, 11008},
                                      {5120, 13824}, {2048, 8192}, {2048, 5632}, {3072, 8192}, {4608, 12288}, {2304, 9216}, {3200, 8640}};
    for (const auto& l : edge_layers)
        for (int64_t M : {(int64_t)1000, momk::long_from(l[0], l[1])}) {
            const momk::Launch a = momk::choose_down(M - 1, l[0], l[1], 256, false), b = momk::choose_down(M, l[0], l[1], 256, false);
            CHECK(a.kind == b.kind && a.tm == b.tm && a.tn == b.tn, "down M=%lld N=%lld K=%lld: %d x %d, one row less %d x %d", (long long)M,
                  (long long)l[0], (long long)l[1], b.tm, b.tn, a.tm, a.tn);
        }
    // What the GPU tests take for granted about the choice: launches of two widths, the second ring of gate/up 64 x 64.
    const int64_t two[][3] = {{1024, 128, 14336}, {1000, 96, 14304}, {2048, 64, 14336}, {1280, 128, 10112}};
    for (const auto& t : two) {
        const momk::Launch l = momk::choose_gateup(t[0], t[2], t[1], 256, false);
        CHECK(l.kind == momk::kTwoWidths && l.wide_cols > 0 && l.wide_cols < t[2], "gate/up M=%lld N=%lld", (long long)t[0], (long long)t[2]);
    }
    const int64_t ring[][3] = {{33, 8192, 7168}, {61, 8192, 7168}, {100, 8192, 3584}};
    for (const auto& t : ring) {
        const momk::Launch l = momk::choose_gateup(t[0], t[2], t[1], 256, false);
        CHECK(l.kind == momk::kShortTiles && l.tm == 64 && l.tn == 64 && l.form != momk::find_short_form(true, 64, 64),
              "gate/up M=%lld N=%lld", (long long)t[0], (long long)t[2]);
    }
    // Down launches of few rows fill the CUs: a short last token tile does not make up for half of them idle (calls of these layers
    // were 4 ... 9 % slower so).
    const int64_t few[][5] = {{57, 2048, 8192, 32, 16}, {64, 2048, 8192, 32, 16}, {58, 2048, 5632, 32, 16}, {64, 2048, 5632, 32, 16},
                              {86, 2048, 8192, 32, 32}, {86, 2560, 9728, 32, 32}, {122, 2048, 8192, 32, 32}, {122, 2048, 5632, 32, 32}};
    for (const auto& t : few) {
        const momk::Launch l = momk::choose_down(t[0], t[1], t[2], 256, false);
        CHECK(l.kind == momk::kShortTiles && l.tm == t[3] && l.tn == t[4], "down M=%lld N=%lld K=%lld in %d x %d", (long long)t[0],
              (long long)t[1], (long long)t[2], l.tm, l.tn);
    }
    // ... and gate/up of 684 ... 768 rows x 9728 columns takes the 228 tiles of 256 x 256 (in 244 of 192 x 320 3 ... 4 % slower).
    for (int64_t M = 684; M <= 768; ++M)
        for (int64_t K : {2560, 3584}) {
            const momk::Launch l = momk::choose_gateup(M, 9728, K, 256, false);
            CHECK(l.kind == momk::kWholeTiles && l.tm == 256 && l.tn == 256, "gate/up M=%lld K=%lld in %d x %d", (long long)M, (long long)K, l.tm, l.tn);
        }
    // Blocks are for mini-sequences of few rows: a layer of 256 x 1024 by 26214 of them and more is faster without.
    for (int64_t C : {128, 512, 9000, 18022, 26214, 32768}) {
        const int64_t S = 2 * C + 3956;
        const momk::Launch g = momk::choose_gateup(C, 1024, 256, 256, true), d = momk::choose_down(C, 256, 1024, 256, false);
        const int form = momk::choose_block(S, 256, 1024, C, 256, g, d);
        CHECK(C > 18022 || form >= 0, "no blocks for mini-sequences of %lld", (long long)C);
        CHECK(C <= 18022 || form < 0, "blocks for mini-sequences of %lld", (long long)C);
    }
    // a form that is not there is an error, not a launch of nothing
    for (bool gu : {false, true})
        for (int f : {-1, momk::short_forms(gu)})
            CHECK(momk::short_launch(100, 256, gu, f).kind == momk::kRefused, "form %d", f);
    int down_form = 0, gateup_form = 0;
#define D(TM, TN, WM, WN, KSUB, NSTG) form(false, down_form++, TM, TN, WM, WN, KSUB, NSTG);
#define G(TM, TN, WM, WN, KSUB, NSTG) form(true, gateup_form++, TM, TN, WM, WN, KSUB, NSTG);
    MOM_SHORT_FORMS_DOWN(D)
    MOM_SHORT_FORMS_GATEUP(G)
    const int64_t Ms[] = {1, 15, 16, 17, 61, 128, 317, 1000, 4096, 131071, 1 << 20, 0x7fffff00};
    const int64_t dims[] = {32, 96, 256, 1056, 3584, 4096, 14336, 18944, 1 << 20};
    int n = 0;
    for (int64_t M : Ms)
        for (int64_t N : dims)
            for (int64_t K : dims)
                for (bool gu : {false, true})
                    for (int cus : {1, 80, 256, 304}) {
                        double cost = -1;
                        const momk::LaunchTime& t = gu ? momk::kShortGateUpTime : momk::kShortDownTime;
                        const int f = momk::choose_short_form(M, N, K, gu, t, cus, cost);
                        ++n;
                        if (f < 0) { CHECK(M > 1 << 20, "no form for M=%lld N=%lld", (long long)M, (long long)N); continue; }
                        CHECK(f < momk::short_forms(gu) && std::isfinite(cost) && cost > 0, "choice");
                        const momk::ShortShape s = momk::short_shape(gu, f);
                        CHECK((int64_t)momk::tile_grid(M, N, gu, s).tiles <= momk::kMaxTiles, "tiles");
                        for (int i = 0; i < momk::short_forms(gu); ++i) {
                            const momk::ShortShape o = momk::short_shape(gu, i);
                            const double c = momk::launch_time(momk::tile_grid(M, N, gu, o), M, K, gu, o, t, cus);
                            CHECK(c < 0 || cost <= c, "least cost: M=%lld N=%lld K=%lld form %d", (long long)M, (long long)N, (long long)K, i);
                        }
                    }
    printf("%d forms, %d choices: %s\n", momk::short_forms(0) + momk::short_forms(1), n, bad ? "FAILED" : "ok");
    return bad != 0;
}

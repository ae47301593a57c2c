// Host check of the short GEMM forms and of the rule that picks one (csrc/mom_gemm_forms.h): what a form assumes
// about its sizes, and that every launch size gets a form that the kernels can run.
#include <cstdio>
#include <cmath>
#include <initializer_list>
#include "mom_gemm_forms.h"

static int bad = 0;
#define CHECK(c, ...) do { if (!(c)) { printf("FAILED %s: ", #c); printf(__VA_ARGS__); printf("\n"); ++bad; } } while (0)

static void form(bool gu, int f, int tm, int tn, int wm, int wn, int ksub, int nstg) {
    const int stage = ksub * (tm + tn) * 128, loads = ksub * (tm + tn) / 32;
    const int cols = gu ? tn / 2 : tn;
    CHECK(nstg * stage <= 163840 && stage <= 65536 && nstg >= 2, "ring of %d x %d", tm, tn);
    CHECK((nstg - 2) * loads <= 63, "loads in flight of %d x %d", tm, tn);
    CHECK(wm * wn <= 4 && tm % (16 * wm) == 0 && tn % (16 * wn) == 0, "wavefront grid of %d x %d", tm, tn);
    CHECK(!gu || (tn / 16 / wn) % 2 == 0, "gate and up blocks of %d x %d", tm, tn);
    CHECK((ksub * tm) % 32 == 0 && (ksub * tn) % (gu ? 64 : 32) == 0, "loads per wavefront of %d x %d", tm, tn);
    CHECK(tm * (cols * 2 + 16) <= nstg * stage, "epilogue of %d x %d", tm, tn);
    const momk::ShortShape s = momk::short_shape(gu, f);
    CHECK(s.tm == tm && s.tn == tn && s.per_cu >= 1 && s.per_cu * nstg * stage <= 163840, "workgroups per CU of %d x %d", tm, tn);
    // Every 1-KiB block of a stage is loaded once, to a place of its own: the kernel's mapping of wavefront and
    // load index to sub-tile and row
    bool seen[2][16][64] = {};                        // [operand][sub][row / 8]
    for (int wave = 0; wave < 4; ++wave)
        for (int j = 0; j < loads; ++j) {
            const int lt = ksub * tm / 32;
            int op, sub, row;
            if (j < lt) {
                const int b = wave + 4 * j;
                op = 0; sub = b / (tm / 8); row = (b % (tm / 8)) * 8;
            } else {
                const int hr = gu ? tn / 2 : tn, w = wave + 4 * (j - lt);
                const int half = w / (ksub * hr / 8), b = w % (ksub * hr / 8);
                op = 1; sub = b / (hr / 8); row = half * hr + (b % (hr / 8)) * 8;
                // the weight matrix is picked by the load index alone
                CHECK(!gu || half == (j - lt >= (loads - lt) / 2), "weight matrix of a load of %d x %d", tm, tn);
            }
            CHECK(sub < ksub && row + 8 <= (op ? tn : tm), "block of %d x %d", tm, tn);
            CHECK(!seen[op][sub][row / 8], "block loaded twice in %d x %d", tm, tn);
            seen[op][sub][row / 8] = true;
        }
}

// The kernels' walk over the tiles of a grid covers every token row once, with a tile of its own for each count that the
// grid states (and that its time was reckoned with): tile i starts at row i tm.
static void rows(int64_t M, int tm, const momk::TileGrid& t) {
    int64_t next = 0;
    for (int64_t i = 0; i < t.tiles_m; ++i) {
        const int64_t m0 = i * tm, end = m0 + (M - m0 < tm ? M - m0 : tm);
        CHECK(m0 == next && m0 < end && m0 <= 0x7fffffff, "tile %lld of M=%lld tm=%d", (long long)i, (long long)M, tm);
        next = end;
    }
    CHECK(next == M, "rows of M=%lld tm=%d", (long long)M, tm);
    CHECK(t.tiles == (uint64_t)t.tiles_m * t.tiles_n, "tiles of M=%lld tm=%d", (long long)M, tm);
}

// What choose_down picks at these sizes, against every launch there is, each priced on the grid that runs.
static int64_t rounds(const momk::TileGrid& g, int cus) { return ((int64_t)g.tiles + cus - 1) / cus; }
static void down_choice(int64_t M, int64_t N, int64_t K, int cus, bool more) {
    const momk::Launch l = momk::choose_down(M, N, K, cus, more, false);
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
        const momk::Launch l = gateup ? momk::choose_gateup(M, N, K, 256) : momk::choose_down(M, N, K, 256, false, false);
        if (M > 1 && same(l, last)) continue;
        CHECK(!since || !same(l, before) || M - since >= 4, "M=%lld N=%lld K=%lld: %d x %d between two runs of %d x %d", (long long)since,
              (long long)N, (long long)K, last.tm, last.tn, l.tm, l.tn);
        before = last;
        last = l;
        since = M;
    }
}

int main() {
    for (int tm = 16; tm <= 256; tm += 16)
        for (int64_t M = 1; M <= 16384; M += 1 + M / 97) rows(M, tm, momk::tile_grid(M, 32, false, {tm, 32, 1, 0}));
    rows(0x7fffff00, 256, momk::tile_grid(0x7fffff00, 32, false, {256, 32, 1, 0}));
    for (int64_t M = 1; M <= 16384; ++M) {
        for (bool more : {false, true}) down_choice(M, 4096, 14336, 256, more);
        for (bool more : {false, true}) down_choice(M, 3584, 18944, 256, more);
        for (bool more : {false, true}) down_choice(M, 8192, 28672, 256, more);
        CHECK(momk::choose_gateup(M, 14336, 4096, 256).kind != momk::kRefused, "gate/up M=%lld", (long long)M);
    }
    const int64_t layers[][2] = {{4096, 14336}, {3584, 18944}, {1056, 2080}, {256, 1024}};
    for (const auto& l : layers) {
        steady(l[0], l[1], false);
        steady(l[1], l[0], true);
    }
    // What the GPU tests take for granted about the choice: launches of two widths, the second ring of gate/up 64 x 64.
    const int64_t two[][3] = {{1024, 128, 14336}, {1000, 96, 14304}, {2048, 64, 14336}, {1280, 128, 10112}};
    for (const auto& t : two) {
        const momk::Launch l = momk::choose_gateup(t[0], t[2], t[1], 256);
        CHECK(l.kind == momk::kTwoWidths && l.wide_cols > 0 && l.wide_cols < t[2], "gate/up M=%lld N=%lld", (long long)t[0], (long long)t[2]);
    }
    const int64_t ring[][3] = {{33, 8192, 7168}, {61, 8192, 7168}, {100, 8192, 3584}};
    for (const auto& t : ring) {
        const momk::Launch l = momk::choose_gateup(t[0], t[2], t[1], 256);
        CHECK(l.kind == momk::kShortTiles && l.tm == 64 && l.tn == 64 && l.form != momk::find_short_form(true, 64, 64),
              "gate/up M=%lld N=%lld", (long long)t[0], (long long)t[2]);
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

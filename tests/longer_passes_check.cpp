// Host check of the passes of more rows than the workspace holds (csrc/mom_gemm_forms.h): every row once, no token tile of the down
// launch in both pieces of the intermediate, and the piece at the end of `out` behind the rows that the pass writes, whatever
// the alignment of `out`.
#include <cstdio>
#include <initializer_list>
#include "mom_gemm_forms.h"

static int bad = 0;
#define CHECK(c, ...) do { if (!(c)) { printf("FAILED %s: ", #c); printf(__VA_ARGS__); printf("\n"); ++bad; } } while (0)

int main() {
    const int64_t layers[][2] = {{4096, 14336}, {3584, 18944}, {1056, 2080}, {256, 1024}, {5120, 25600}, {2048, 8192}, {8192, 28672}, {1024, 1024}, {4096, 32}, {32, 32}};
    int calls = 0, longer = 0, split = 0, whole = 0;
    for (const auto& l : layers)
        for (int64_t C = 1; C < 20000; C += 1 + C * 3 / 7)
            for (int64_t S : {C + 1, 2 * C, 3 * C + C / 3, 6 * C + 5, 16 * C, 64 * C + 7, 300 * C + 1}) {
                const int64_t H = l[0], I = l[1];
                if (!momk::longer_passes(S, H, I, C)) continue;
                momk::Passes passes(S, H, I, C, 256, true);
                int64_t r0 = 0;
                ++calls;
                for (int n = 0; r0 < S && n < 400; ++n) {
                    const int64_t left = S - r0;
                    const momk::Pass p = passes.next();
                    CHECK(passes.left == left && p.rows > 0 && p.rows <= left, "left");
                    passes.done(p);
                    if (p.split == momk::kWhole) { CHECK(p.rows == (left < C ? left : C), "rows"); r0 += p.rows; continue; }
                    ++longer;
                    (p.split ? split : whole) += 1;
                    CHECK(p.rows > C && p.rows < left && p.rows % 256 == 0, "rows S=%lld C=%lld H=%lld", (long long)S, (long long)C, (long long)H);
                    CHECK(p.split >= 0 && p.split <= C && p.split % p.down.tm == 0, "split %lld of C=%lld, tiles of %d", (long long)p.split, (long long)C, p.down.tm);
                    CHECK(p.gateup.kind != momk::kRefused && p.down.kind != momk::kRefused, "launches");
                    for (int64_t out : {0, 16, 112, 240, 256}) {        // address of `out`, bytes
                        const int64_t end = out + S * H * 2, at = (end - (p.rows - p.split) * I * 2) & ~(momk::kSpareAlign - 1);
                        CHECK(at >= out + (r0 + p.rows) * H * 2, "rows %lld at %lld of S=%lld C=%lld H=%lld I=%lld", (long long)p.rows, (long long)r0,
                              (long long)S, (long long)C, (long long)H, (long long)I);
                        CHECK(at + (p.rows - p.split) * I * 2 <= end, "end");
                    }
                    r0 += p.rows;
                }
            }
    CHECK(longer > 1000 && split > 300 && whole > 100, "%d longer passes, %d split, %d whole", longer, split, whole);
    // what was measured: calls that take fewer passes, and one that has none to take
    // (the first two: the first passes of a call don't find W_down in the cache, a longer one is weighed against what they take)
    const int64_t fewer[][5] = {{3077, 3584, 18944, 512, 768}, {4096, 3584, 18944, 512, 1024}, {8192, 4096, 14336, 512, 2048}, {16384, 4096, 14336, 256, 3328}, {8197, 1056, 2080, 512, 2816}};
    for (const auto& t : fewer) {
        const momk::Pass p = momk::Passes(t[0], t[1], t[2], t[3], 256, true).next();
        CHECK(p.rows == t[4], "S=%lld C=%lld: %lld rows, not %lld", (long long)t[0], (long long)t[3], (long long)p.rows, (long long)t[4]);
    }
    // ... and calls that longer passes made slower: as many passes, of lengths that take as long or longer
    const int64_t none[][4] = {{3072, 512, 1536, 1024}, {3072, 1024, 4096, 1024}, {7471, 512, 1536, 2500}, {2328, 1056, 2080, 1280}, {3361, 1056, 2080, 1280},
                               {2494, 1056, 2080, 1280}, {3000, 1056, 2080, 1600}, {3000, 1056, 2080, 1024}, {2084, 1024, 4096, 800}, {2939, 1056, 2080, 1500},
                               {1000, 1056, 2080, 200}};
    for (const auto& t : none) {
        momk::Passes passes(t[0], t[1], t[2], t[3], 256, true);
        while (passes.left > 0) {
            const momk::Pass p = passes.next();
            CHECK(p.split == momk::kWhole, "S=%lld C=%lld H=%lld: %lld rows", (long long)t[0], (long long)t[3], (long long)t[1], (long long)p.rows);
            passes.done(p);
        }
    }
    CHECK(!momk::longer_passes(32768, 4096, 14336, 4096) && !momk::longer_passes(300, 256, 1024, 100) && !momk::longer_passes(512, 4096, 14336, 512), "asked for");
    // What blocks are weighed against is what the driver runs: calls in blocks of several rounds of the CUs take no more than its passes would.
    int blocks = 0, instead = 0;
    for (int64_t C : {128, 181, 256, 300, 512, 1024})
        for (int64_t S = 4100; S < 24000; S += 37) {
            const int64_t H = 1056, I = 2080;
            momk::Passes passes(S, H, I, C, 256, true);
            const momk::Pass p = passes.plain();
            const double expected = passes.time();
            double t = 0;
            while (passes.left > 0) { const momk::Pass q = passes.next(); t += q.time(); passes.done(q); }
            CHECK(t > 0.9999 * expected && t < 1.0001 * expected, "S=%lld C=%lld: %.1f us, by pass %.1f", (long long)S, (long long)C, expected, t);
            const int form = momk::choose_block(S, H, I, C, 256, p.gateup, p.down);
            if (form < 0) { ++instead; continue; }
            ++blocks;
            const double b = momk::block_time(momk::kBlockForms[form], S, H, I, 256);
            CHECK(b <= 1.02 * t || momk::block_count(momk::kBlockForms[form], S) <= 256, "S=%lld C=%lld in blocks: %.1f us, passes %.1f", (long long)S, (long long)C, b, t);
        }
    CHECK(instead > 1000, "%d calls in blocks, %d in passes", blocks, instead);
    printf("%d calls, %d longer passes: %s\n", calls, longer, bad ? "FAILED" : "ok");
    return bad != 0;
}

// Host check of the shares of a block's output columns (csrc/mom_gemm_forms.h): every group of 32 columns in one workgroup, none of them empty, and
// no more workgroups than CUs where there are shares.
#include <cstdio>
#include "mom_gemm_forms.h"

int main() {
    int bad = 0, shared = 0;
    for (const momk::BlockForm& f : momk::kBlockForms)
        for (int cus : {1, 80, 256, 304})
            for (int64_t H = 32; H <= 8192; H += 32)
                for (int64_t S = 1; S < 40000; S += 1 + S / 5) {
                    const uint32_t blocks = momk::block_count(f, S);
                    const int64_t groups = H / 32;
                    const int share = momk::block_share(blocks, H, cus);
                    const int64_t parts = momk::block_parts(H, share);
                    const bool ok = (int64_t)blocks * 16 * f.tb >= S && share >= 1 && parts >= 1 && parts <= 8 && (parts - 1) * share < groups &&
                                    parts * share >= groups && (parts == 1 || (share >= 4 && (int64_t)blocks * parts <= cus));
                    shared += parts > 1;
                    if (!ok) { printf("FAILED S=%lld H=%lld cus=%d: %lld parts of %d\n", (long long)S, (long long)H, cus, (long long)parts, share); if (++bad > 20) return 1; }
                }
    printf("%d shared: %s\n", shared, bad || shared < 10000 ? "FAILED" : "ok");
    return bad || shared < 10000;
}

// Host-only probe of the choice of kernels for forward solves: reads problems "G S PR kind dtype B L H fixed" from stdin (fixed:
// iterations of a solve of a fixed count, 0 = to a tolerance) and prints one line each: 0 with carry records, 1 one
// workgroup per channel group, 2 waves that walk (walk_kernels.h); then steps per thread, log2 of the channels per group, waves,
// workgroups, tiles, polls of the wait for the verdicts.  No device call.
#include <stdio.h>

#include "pararnn/driver.h"

using namespace pararnn;

int main()
{
    int G, S, PR, kind, dtype, B, L, H, fixed;
    while (scanf("%d %d %d %d %d %d %d %d %d", &G, &S, &PR, &kind, &dtype, &B, &L, &H, &fixed) == 9) {
        const CellInfo ci = {G, S, PR, kind};
        const SolveOpts opts = {1, kFusedHead, false};
        const ShortShape none = {-1, -1, -1, -1, -1, -1};
        ShortShape sh = none;
        const bool found = without_blocks(ci, dtype, B, L, H, fixed ? -1.0f : 1e-5f, fixed ? fixed : 64, opts, &sh);
        if (!found) {
            if (sh.c != none.c || sh.lps_log2 != none.lps_log2 || sh.w != none.w || sh.n_items != none.n_items) {
                fprintf(stderr, "a shape without a choice\n");
                return 1;
            }
            sh = ShortShape{};
        }
        printf("%d %d %d %d %d %d %u\n", found ? sh.walk ? 2 : 1 : 0, sh.c, sh.lps_log2, sh.w, sh.n_items, sh.n_tiles,
               found ? short_wait_limit(kSpinLimit, sh, fixed ? fixed : 64) : 0);
    }
    return 0;
}

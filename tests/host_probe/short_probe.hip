// Host-only probe of the choice between the kernels that keep a channel group in one workgroup (short_kernels.h) and
// those with carry records: reads problems "G S PR kind dtype B L H backward fixed" from stdin (fixed: iterations of a
// solve of a fixed count, 0 = to a tolerance) and prints one line each: steps per thread, log2 of the channels per
// group, waves, workgroups, tiles, polls of the wait for the verdicts; zeros where the kernels with records are taken.  No device call.
#include <stdio.h>

#include "pararnn/driver.h"

using namespace pararnn;

int main()
{
    int G, S, PR, kind, dtype, B, L, H, backward, fixed;
    while (scanf("%d %d %d %d %d %d %d %d %d %d", &G, &S, &PR, &kind, &dtype, &B, &L, &H, &backward, &fixed) == 10) {
        const CellInfo ci = {G, S, PR, kind};
        ShortShape sh = {};
        if (!short_shape(ci, dtype, B, L, H, backward != 0, fixed, &sh)) sh = ShortShape{};
        const unsigned int polls = sh.c ? short_wait_limit(kSpinLimit, sh, fixed ? fixed : 64) : 0;
        printf("%d %d %d %d %d %u\n", sh.c, sh.lps_log2, sh.w, sh.n_items, sh.n_tiles, polls);
    }
    return 0;
}

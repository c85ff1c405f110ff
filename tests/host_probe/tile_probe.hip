// Host-only probe of the tile of a backward pass with carry records: reads problems "G S PR kind dtype B L H" from stdin and
// prints one line each: the shape that choose_tile's table has, the one that is taken, and whether rows are staged where
// they can be.  No device call.
#include <stdio.h>

#include "pararnn/driver.h"

using namespace pararnn;

int main()
{
    int G, S, PR, kind, dtype, B, L, H;
    while (scanf("%d %d %d %d %d %d %d %d", &G, &S, &PR, &kind, &dtype, &B, &L, &H) == 8) {
        const CellInfo ci = {G, S, PR, kind};
        const TileCfg t = choose_tile(ci, dtype, true, H, 4, false);
        const TileCfg n = make_layout(ci, dtype, B, L, H, true, 4).cfg;
        printf("%d %d %d %d %d %d %d %d %d\n", t.vec, t.ll, t.c, t.w, n.vec, n.ll, n.c, n.w, (int)backward_staged(ci, B, L, H));
    }
    return 0;
}

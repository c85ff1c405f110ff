// Host-only probe of the tile of a backward pass with carry records: reads problems "G S PR kind dtype B L H" from stdin and
// prints one line each: the shape that choose_tile's table has, the one that is taken, whether rows are staged where
// they can be, whether there is a queue of tiles for each XCD, the shape of a forward solve's blocks with records, and the
// one that a workspace of 32 MiB holds (zeros: none).  No device call.
#include <stdio.h>

#include "pararnn/driver.h"

using namespace pararnn;

int main()
{
    int G, S, PR, kind, dtype, B, L, H;
    while (scanf("%d %d %d %d %d %d %d %d", &G, &S, &PR, &kind, &dtype, &B, &L, &H) == 8) {
        const CellInfo ci = {G, S, PR, kind};
        const TileCfg t = choose_tile(ci, dtype, true, H, 4, false);
        const Layout lo = make_layout(ci, dtype, B, L, H, true, 4);
        const TileCfg &n = lo.cfg;
        const size_t bytes = (size_t)B * L * H * (dtype == PARARNN_BF16 ? 2 : 4) * (2 * G + 2 * S);
        const TileCfg f = make_layout(ci, dtype, B, L, H, false, 4, true, 5).cfg;
        Layout in;
        if (!fused_layout(ci, dtype, B, L, H, 4, 5, true, [](const Layout &, size_t whole) { return whole <= (size_t)32 << 20; }, &in)) in.cfg = TileCfg{0, 0, 0, 0};
        printf("%d %d %d %d %d %d %d %d %d %d %d %d %d %d %d %d %d %d\n", t.vec, t.ll, t.c, t.w, n.vec, n.ll, n.c, n.w, (int)backward_staged(ci, B, L, H),
               (int)backward_queues(ci, dtype, bytes, lo.g, n), f.vec, f.ll, f.c, f.w, in.cfg.vec, in.cfg.ll, in.cfg.c, in.cfg.w);
    }
    return 0;
}

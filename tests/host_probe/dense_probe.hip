// Host-only probe of the choice between chunk products and forward substitution of the dense cell: reads problems "B L backward"
// from stdin and prints one line each: stretches of a sequence (0: chunk products), steps of a stretch.  No device call.
#include <stdio.h>

#include "dense_plan.h"

int main()
{
    int B, L, backward;
    while (scanf("%d %d %d", &B, &L, &backward) == 3) {
        const pararnn::DensePlan p = pararnn::wavefront_plan(B, L, backward != 0);
        printf("%d %d\n", p.n, p.len);
    }
    return 0;
}

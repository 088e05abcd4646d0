// Evaluates the rules that pick a launch's shape (paper_2605_28691_amd/csrc/wg_shape.h) on the host.  Reads calls from stdin, one a line:
// launch (fwd or bwd), head_dim, B, heads, T, H, W, s, group, pad; prints the number of the shape of each.  A launch named "rows" has the
// bytes of a row in place of head_dim and prints the rows that a wavefront moves; "fp8" prints 1 where the 8-bit kernel of the any-resolution mode
// starts every tile's logits at the keys' bias, "chain" prints 1 where the backward is one walk if it has the workspace, "kernel" the forward kernel that the shape of "fwd" runs in.  Built and run by tests/test_wg_shape.py.
#include <cstdio>
#include <cstring>

#include "../paper_2605_28691_amd/csrc/kernels.h"

using namespace skiparse;

int main() {
    char launch[8];
    int D, B, heads, T, H, W, s, group, pad;
    while (scanf("%7s %d %d %d %d %d %d %d %d %d", launch, &D, &B, &heads, &T, &H, &W, &s, &group, &pad) == 10) {
        if (strcmp(launch, "rows") == 0) {
            printf("%u\n", row_batch((uint32_t)(D / 16), (uint32_t)(B * T * H * W)));
            continue;
        }
        const GridMap g = make_gridmap(T, H, W, s, group != 0, pad != 0);
        const UnitSizes u = unit_sizes(g, pad != 0 && s > 1, (uint64_t)B * (uint64_t)heads);
        if (strcmp(launch, "fp8") == 0) printf("%d\n", pads_most_tiles(D, g) ? 1 : 0);
        else if (strcmp(launch, "chain") == 0) printf("%d\n", bwd_chain(D, u) ? 1 : 0);
        else if (strcmp(launch, "kernel") == 0) printf("%d\n", fwd_kernel(D, pad != 0 && s > 1, u));
        else printf("%d\n", strcmp(launch, "fwd") == 0 ? pick_fwd_shape(D, u) : pick_bwd_shape(D, u));
    }
    return 0;
}

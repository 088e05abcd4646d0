// Evaluates the rules that pick a launch's shape (paper_2605_28691_amd/csrc/wg_shape.h) on the host.  Reads calls from stdin, one a line:
// launch (fwd or bwd), head_dim, B, heads, T, H, W, s, group, pad; prints the number of the shape of each.  A launch named "rows" has the
// bytes of a row in place of head_dim and prints the rows that a wavefront moves; "fp8" prints 1 where the 8-bit kernel of the any-resolution mode
// starts every tile's logits at the keys' bias, "chain" prints 1 where the backward is one walk if it has the workspace, "queue" the
// units that its queue hands out at a time, or 0 where that does not hand out every block of every unit once and behind the one in front of it, "kernel" the forward kernel that the shape of "fwd" runs in.  Built and run by tests/test_wg_shape.py.
#include <cstdio>
#include <cstring>
#include <vector>

#include "../paper_2605_28691_amd/csrc/kernels.h"

using namespace skiparse;

// The tickets of attn_bwd_chain.hip's workgroups, drawn one after the other by those of `xccs` XCCs in an order that goes by `seed`.
static bool hands_out_all(const BwdChain& w, uint32_t xccs, uint32_t seed) {
    constexpr uint32_t WORKGROUPS = 32;  // of an XCC
    std::vector<uint32_t> tickets(xccs), refused(xccs), slots(xccs * (w.n_units + 1u)), next(w.n_units), on(w.n_units);
    uint32_t groups = 0, left = xccs;
    while (left != 0) {
        seed = seed * 1664525u + 1013904223u;
        const uint32_t x = (seed >> 8) % xccs;
        if (refused[x] == WORKGROUPS) continue;
        const uint32_t n = tickets[x]++, g = n / w.per_group, r = n % w.per_group;
        uint32_t task = CHAIN_NONE;
        if (g <= w.n_groups) {
            if (g > w.n_units) return false;  // as many slots as units and one
            uint32_t& id = slots[x * (w.n_units + 1u) + g];
            if (r == 0) id = ++groups;
            task = w.task(id, r);
        }
        if (task == CHAIN_SKIP) continue;
        if (task == CHAIN_NONE) {
            left -= ++refused[x] == WORKGROUPS;
            continue;
        }
        const uint32_t unit = task / w.n_blk, blk = task % w.n_blk;
        if (unit >= w.n_units || blk != next[unit]++ || (blk != 0 && on[unit] != x)) return false;
        on[unit] = x;
    }
    for (uint32_t blocks : next)
        if (blocks != w.n_blk) return false;
    return true;
}

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
        else if (strcmp(launch, "queue") == 0) {
            const BwdChain w = make_bwd_chain((uint32_t)(B * heads) * (g.mode == MODE_DENSE ? 1u : (uint32_t)(s * s)), u.n_max);
            printf("%u\n", hands_out_all(w, XCDS, 1) && hands_out_all(w, XCDS, 2) && hands_out_all(w, 1, 3) && hands_out_all(w, CHAIN_XCCS, 4) ? w.together : 0u);
        }
        else if (strcmp(launch, "kernel") == 0) printf("%d\n", fwd_kernel(D, pad != 0 && s > 1, u));
        else printf("%d\n", strcmp(launch, "fwd") == 0 ? pick_fwd_shape(D, u) : pick_bwd_shape(D, u));
    }
    return 0;
}

// Host-side check of the row moves: source_row() of every destination row against the plain formulas of Algorithm 1 (both patterns, all three
// directions, and the receive buffers of Sparse Sequence Parallelism against the axis swap they stand for), Div32 at the edges of every
// quotient, and the parts of a row: they cover it once, in whole lines, within the size of a grid.  Built and run by tests/test_host_logic.py.
#include <cstdio>
#include <vector>

#include "../paper_2605_28691_amd/csrc/kernels.h"

using namespace skiparse;

// row of token (b, t, h, w) in the sparse layout of a pattern
static uint32_t sparse_row(bool group, int B, int T, int H, int W, int s, int b, int t, int h, int w) {
    const int p = group ? (h / s) % s : h % s, q = group ? (w / s) % s : w % s;
    const int hs = group ? h / (s * s) * s + h % s : h / s, ws = group ? w / (s * s) * s + w % s : w / s;
    return (uint32_t)((((p * s + q) * B + b) * T + t) * (H / s) + hs) * (uint32_t)(W / s) + (uint32_t)ws;
}

int main() {
    long checked = 0;
    const int shapes[][5] = {{1, 2, 8, 8, 2}, {2, 3, 8, 12, 2}, {1, 2, 9, 18, 3}, {3, 1, 16, 32, 4}, {1, 21, 48, 80, 2}, {2, 2, 3, 5, 1}, {1, 1, 25, 50, 5}, {3, 5, 30, 52, 2}, {1, 1, 1, 4, 1}};
    for (auto& sh : shapes) {
        const int B = sh[0], T = sh[1], H = sh[2], W = sh[3], s = sh[4];
        for (int group = 0; group < 2; group++) {
            if (H % s || W % s || (group && (H % (s * s) || W % (s * s)))) continue;
            const GridMap g = make_gridmap(T, H, W, s, group != 0);
            const RowArgs to = make_row_args<TO_SPARSE>(g, (uint32_t)B), back = make_row_args<TO_ORIGINAL>(g, (uint32_t)B), sw = make_row_args<SWITCH>(g, (uint32_t)B);
            const bool both = H % (s * s) == 0 && W % (s * s) == 0 && s > 1;
            for (int b = 0; b < B; b++)
                for (int t = 0; t < T; t++)
                    for (int h = 0; h < H; h++)
                        for (int w = 0; w < W; w++) {
                            const uint32_t orig = (uint32_t)(((b * T + t) * H + h) * W + w);
                            const uint32_t mine = s == 1 ? orig : sparse_row(group != 0, B, T, H, W, s, b, t, h, w);
                            bool ok = source_row<TO_SPARSE>(to, mine, 0u) == orig && source_row<TO_ORIGINAL>(back, orig, 0u) == mine;
                            if (both) ok = ok && source_row<SWITCH>(sw, mine, 0u) == sparse_row(group == 0, B, T, H, W, s, b, t, h, w);
                            if (!ok) {
                                printf("row mismatch B%d T%d H%d W%d s%d group%d at b%d t%d h%d w%d\n", B, T, H, W, s, group, b, t, h, w);
                                return 1;
                            }
                            checked++;
                        }
        }
        // receive buffer [source rank][g'][g][b][position]: the token-wise split of G*b batch elements with the two subsequence axes swapped
        if (H % s || W % s || s == 1) continue;
        for (int ranks = 1; ranks <= s * s; ranks++) {
            if (s * s % ranks) continue;
            const int G = s * s / ranks, Bl = G * B;
            const GridMap g = make_gridmap(T, H, W, s, false);
            const RowArgs back = make_row_args<TO_ORIGINAL>(g, (uint32_t)Bl);
            for (int gd = 0; gd < G; gd++)
                for (int b = 0; b < B; b++)
                    for (uint32_t n = 0; n < (uint32_t)g.n_tok; n++) {
                        const int w = (int)n % W, h = (int)n / W % H, t = (int)n / (W * H), bl = gd * B + b;
                        const uint32_t plain = sparse_row(false, Bl, T, H, W, s, bl, t, h, w), pq = plain / (uint32_t)(Bl * g.n_sub), j = plain % (uint32_t)g.n_sub;
                        const uint32_t r = pq / G, gs = pq % G, sb = ((r * G + gd) * G + gs) * B + b;
                        if (source_row<TO_ORIGINAL>(back, (uint32_t)bl * (uint32_t)g.n_tok + n, (uint32_t)G) != sb * (uint32_t)g.n_sub + j) {
                            printf("receive buffer mismatch T%d H%d W%d s%d ranks%d token %u\n", T, H, W, s, ranks, n);
                            return 1;
                        }
                        checked++;
                    }
        }
    }
    for (uint32_t d : {1u, 2u, 3u, 5u, 7u, 10u, 64u, 641u, 65535u, 65536u, 80640u, 0x7fffffffu, 0x80000000u, 0xfffffffeu, 0xffffffffu}) {
        const Div32 f = make_div32(d);
        const uint32_t top = 0xffffffffu / d;
        for (uint64_t k = 0; k <= top; k += (top > 2000000u ? top / 999983u : 1u))
            for (uint64_t n : {k * d, k * d + 1u, k * d + d - 1u, k * d + d / 2u}) {
                if (n > 0xffffffffull) continue;
                if (f.div((uint32_t)n) != (uint32_t)n / d) { printf("Div32 %u fails at %llu\n", d, (unsigned long long)n); return 1; }
                checked++;
            }
        for (uint32_t back = 0; back < 1000; back++)
            if (f.div(0xffffffffu - back) != (0xffffffffu - back) / d) { printf("Div32 %u fails at the top\n", d); return 1; }
    }
    for (uint32_t n_rows : {1u, 80640u, 1u << 20, 1u << 25, 1u << 26, 0x7fffffffu})
        for (uint32_t chunks = 1; chunks < 5000; chunks++) {
            const uint32_t u = row_unroll(chunks), span = row_span(chunks, n_rows, u), parts = (chunks + span - 1u) / span;
            const bool one_round = span <= 64u * u || (uint64_t)n_rows * ((chunks + 64u * u - 1u) / (64u * u)) > MAX_ROW_WAVES;
            if (span % 8u || (uint64_t)span * (parts - 1u) >= chunks || (parts > 1u && (uint64_t)n_rows * parts > MAX_ROW_WAVES) || !one_round) {
                printf("parts of %u chunks, %u rows: %u of %u\n", chunks, n_rows, parts, span);
                return 1;
            }
            checked++;
        }
    printf("ok %ld checks\n", checked);
    return 0;
}

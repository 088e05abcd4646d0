// Host-side check of the device index map (paper_2605_28691_amd/csrc/index_map.h): src_token() with its multiply-high
// divisions must equal the plain integer formulas of Algorithm 1 for every position of a grid, and src_token_padded() (the
// any-resolution map, Sec. 3.2) the plain pad-then-index formulas on grids that are not multiples of s*s;
// src_token_real() must enumerate exactly the real positions of src_token_padded(), in their order.  Built and run by
// tests/test_host_logic.py with hipcc (host pass only); exits non-zero on the first mismatch.
#include <cstdio>
#include <cstdlib>

#include "../paper_2605_28691_amd/csrc/index_map.h"

using namespace skiparse;

int main() {
    const int shapes[][4] = {{2, 8, 8, 2}, {3, 8, 12, 2}, {21, 48, 80, 2}, {2, 9, 18, 3}, {1, 16, 32, 4}, {5, 2, 2, 2}, {3, 4, 4, 2}, {1, 25, 50, 5}, {21, 30, 52, 2}};
    long checked = 0;
    for (auto& sh : shapes) {
        const int T = sh[0], H = sh[1], W = sh[2], s = sh[3];
        for (int group = 0; group < 2; group++) {
            if (group && (H % (s * s) || W % (s * s))) continue;
            const GridMap g = make_gridmap(T, H, W, s, group != 0);
            const int Hs = H / s, Ws = W / s;
            for (int p = 0; p < s; p++)
                for (int q = 0; q < s; q++)
                    for (int j = 0; j < g.n_sub; j++) {
                        const int ws = j % Ws, hs = (j / Ws) % Hs, t = j / (Ws * Hs);
                        const int h = group ? (hs / s) * s * s + p * s + hs % s : hs * s + p;
                        const int w = group ? (ws / s) * s * s + q * s + ws % s : ws * s + q;
                        const uint32_t want = (uint32_t)((t * H + h) * W + w);
                        const uint32_t got = src_token(g, (uint32_t)p, (uint32_t)q, (uint32_t)j);
                        if (got != want) {
                            printf("mismatch T%d H%d W%d s%d group%d p%d q%d j%d: got %u want %u\n", T, H, W, s, group, p, q, j, got, want);
                            return 1;
                        }
                        checked++;
                    }
        }
    }
    // any-resolution mode (Sec. 3.2): pad the END of H and W to multiples of s*s, index the padded grid with Algorithm 1's
    // formulas, and call a position real when it lies inside the unpadded grid; its token number is then counted on the
    // unpadded grid.  Every real token must be met exactly once over all classes.
    const int pad_shapes[][4] = {{2, 7, 9, 2}, {3, 5, 6, 2}, {1, 10, 11, 3}, {2, 3, 3, 2}, {1, 17, 13, 4}, {4, 8, 10, 2}, {2, 9, 9, 3}, {21, 45, 80, 2}, {3, 8, 8, 2}, {2, 1, 1, 3}, {1, 2, 33, 4}, {3, 16, 17, 4}};
    for (auto& sh : pad_shapes) {
        const int T = sh[0], H = sh[1], W = sh[2], s = sh[3];
        const int Hp = (H + s * s - 1) / (s * s) * (s * s), Wp = (W + s * s - 1) / (s * s) * (s * s);
        for (int group = 0; group < 2; group++) {
            const GridMap g = make_gridmap(T, H, W, s, group != 0, true);
            if (g.n_sub != T * Hp * Wp / (s * s) || g.n_tok != T * H * W) { printf("padded sizes wrong\n"); return 1; }
            const int Hs = Hp / s, Ws = Wp / s;
            long n_real = 0;
            unsigned char* seen = (unsigned char*)calloc((size_t)T * H * W, 1);
            for (int p = 0; p < s; p++)
                for (int q = 0; q < s; q++)
                    for (int j = 0; j < g.n_sub; j++) {
                        const int ws = j % Ws, hs = (j / Ws) % Hs, t = j / (Ws * Hs);
                        const int h = group ? (hs / s) * s * s + p * s + hs % s : hs * s + p;
                        const int w = group ? (ws / s) * s * s + q * s + ws % s : ws * s + q;
                        const bool want_real = h < H && w < W;
                        bool real = false;
                        const uint32_t got = src_token_padded(g, (uint32_t)p, (uint32_t)q, (uint32_t)j, &real);
                        if (real != want_real || (want_real && got != (uint32_t)((t * H + h) * W + w))) {
                            printf("padded mismatch T%d H%d W%d s%d group%d p%d q%d j%d: got %u real %d, want real %d\n", T, H, W, s, group, p, q, j, got, (int)real, (int)want_real);
                            return 1;
                        }
                        if (real) {
                            if (seen[got]++) { printf("padded map meets token %u twice\n", got); return 1; }
                            n_real++;
                        }
                        checked++;
                    }
            // the real positions of a class as a dense sequence: the same tokens in the same order, and the padded positions they stand for
            for (int p = 0; p < s; p++)
                for (int q = 0; q < s; q++) {
                    const ClassMap c = make_class_map(g, (uint32_t)p, (uint32_t)q);
                    uint32_t k = 0;
                    for (int j = 0; j < g.n_sub; j++) {
                        bool real = false;
                        const uint32_t tok = src_token_padded(g, (uint32_t)p, (uint32_t)q, (uint32_t)j, &real);
                        if (!real) continue;
                        if (k >= c.n || src_token_real(g, c, (uint32_t)p, (uint32_t)q, k) != tok || padded_position(g, c, k) != (uint32_t)j) {
                            printf("dense map mismatch T%d H%d W%d s%d group%d p%d q%d position %u\n", T, H, W, s, group, p, q, k);
                            return 1;
                        }
                        k++;
                        checked++;
                    }
                    // rows and columns of the class, as selected from what the host hands to the kernels
                    uint32_t rows = 0, cols = 0;
                    for (int h = 0; h < H; h++) rows += (group ? h / s : h) % s == p;
                    for (int w = 0; w < W; w++) cols += (group ? w / s : w) % s == q;
                    if (c.h.d != rows || c.w.d != cols || c.hs.d != (uint32_t)Hs) {
                        printf("class extents T%d H%d W%d s%d group%d p%d q%d\n", T, H, W, s, group, p, q);
                        return 1;
                    }
                    if (k != c.n || c.n > make_class_map(g, 0, 0).n || c.n < make_class_map(g, (uint32_t)s - 1, (uint32_t)s - 1).n) {
                        printf("dense map: class %d %d has %u real tokens, the map says %u\n", p, q, k, c.n);
                        return 1;
                    }
                }
            free(seen);
            if (n_real != (long)T * H * W) { printf("padded map: %ld real positions, want %d\n", n_real, T * H * W); return 1; }
        }
    }
    // the multiply-high division over its whole admissible range for a few divisors: n * d < 2^32
    for (uint32_t d : {1u, 2u, 3u, 7u, 40u, 64u, 641u, 65535u}) {
        for (int narrow = 0; narrow < 2; narrow++) {
        const FastDiv f = narrow ? make_fastdiv32(d) : make_fastdiv(d);
        const uint64_t limit = (1ull << 32) / d;
        for (uint64_t n = 0; n < limit; n += (limit > 5000000 ? limit / 4999999 : 1)) {
            if (f.div((uint32_t)n) != (uint32_t)(n / d)) { printf("fastdiv %u fails at %llu\n", d, (unsigned long long)n); return 1; }
            checked++;
        }
        const uint32_t last = (uint32_t)(limit - 1);
        if (f.div(last) != last / d) { printf("fastdiv %u fails at the top of its range\n", d); return 1; }
        }
    }
    // the number of a workgroup taken apart as integer divisions do it, both orders of the units
    for (uint32_t tiles : {1u, 3u, 79u, 158u})
        for (uint32_t B : {1u, 2u, 36u})
            for (uint32_t heads : {1u, 5u, 40u})
                for (uint32_t s : {1u, 2u, 3u}) {
                    GridMap g = s == 1 ? make_dense_gridmap(10) : make_gridmap(1, 2 * (int)(s * s), 2 * (int)(s * s), (int)s, false);
                    const UnitMap by_unit = make_unit_map<false>(g, tiles, B, heads), by_head = make_unit_map<true>(g, tiles, B, heads);
                    for (uint32_t lin = 0; lin < tiles * B * s * s * heads; lin++) {
                        const uint32_t unit = lin / tiles, n_bb = B * s * s;
                        const UnitAt a = by_unit.at<false>(lin), h = by_head.at<true>(lin);
                        const bool ok = a.unit == unit && a.tile == lin % tiles && a.bb == unit / heads && a.head == unit % heads && a.p == unit / heads / B / s && a.q == unit / heads / B % s &&
                                        a.b == unit / heads % B && h.unit == unit && h.tile == lin % tiles && h.head == unit / n_bb && h.bb == unit % n_bb && h.p == unit % n_bb / B / s &&
                                        h.q == unit % n_bb / B % s && h.b == unit % n_bb % B;
                        if (!ok) { printf("unit map: tiles %u B %u heads %u s %u workgroup %u\n", tiles, B, heads, s, lin); return 1; }
                        checked++;
                    }
                }
    printf("ok %ld checks\n", checked);
    return 0;
}

// Skiparse index maps for device code (Algorithm 1, "Skiparse Rearrange").
//
// A subsequence is named by its spatial class (p, q) and a batch element b; position j inside it enumerates
// (t, hs, ws) row-major over the reduced grid (T, H/s, W/s).  src_token() returns the token number
// n = (t*H + h)*W + w that sits at position j.  Because t*H + h and hs only ever appear combined, the map needs a
// single division of j by W/s:
//     r = j / Ws (= t*Hs + hs),  ws = j % Ws
//     token-wise: t*H + h = r*s + p                      w = ws*s + q
//     group-wise: t*H + h = (r/s)*s*s + p*s + r%s        w = (ws/s)*s*s + q*s + ws%s     (needs Hs % s == 0)
// Both are instances of one branch-free form  f(x) = x*a + (x/s)*b + c  with (a, b) = (s, 0) for token-wise and
// (1, s*s - s) for group-wise, c = p (or q) for token-wise and p*s (or q*s) for group-wise.  The dense case (position j is
// token j) uses a = 1, b = 0, c = 0 and a divisor of 2^31 so that r is always 0.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace skiparse {

enum Mode : int { MODE_DENSE = 0, MODE_TOKEN = 1, MODE_GROUP = 2 };

// Division of a 32-bit n by a run-time constant d through one multiply-high; exact while n * d < 2^32
// (mul = floor(2^32 / d) + 1, so mul * d = 2^32 + e with 1 <= e <= d and the error term n * e / 2^32 stays below 1).
// d = 1 would need a multiplier of 2^32: it is expressed as mul = 0 plus `one` = 1 (quotient = n * one).
struct FastDiv {
    uint32_t d;
    uint32_t mul;
    uint32_t one;
    __host__ __device__ inline uint32_t div(uint32_t n) const {
#if defined(__HIP_DEVICE_COMPILE__)
        return __umulhi(n, mul) + n * one;
#else
        return (uint32_t)(((uint64_t)n * mul) >> 32) + n * one;
#endif
    }
};

inline FastDiv make_fastdiv(uint32_t d) {
    FastDiv f;
    f.d = d;
    f.mul = d <= 1u ? 0u : (uint32_t)((1ull << 32) / d) + 1u;
    f.one = d <= 1u ? 1u : 0u;
    return f;
}

// make_fastdiv in 32-bit arithmetic: the same multiplier except at powers of two, where 2^32 / d is exact (e = 0)
__host__ __device__ inline FastDiv make_fastdiv32(uint32_t d) {
    FastDiv f;
    f.d = d;
    f.mul = d <= 1u ? 0u : 0xffffffffu / d + 1u;
    f.one = d <= 1u ? 1u : 0u;
    return f;
}

struct GridMap {
    int mode;      // MODE_DENSE: position j is token j
    int s;         // sparse ratio
    int W;         // original row length
    int n_tok;     // tokens per batch element in the original layout (T*H*W)
    int n_sub;     // tokens per subsequence
    int T;         // frames
    uint32_t a;    // f(x) = x*a + (x/s)*b + c, see above
    uint32_t b;
    uint32_t cmul; // c = p*cmul (rows) or q*cmul (columns)
    FastDiv ws;    // division by W/s
    FastDiv sdiv;  // division by s
    // Any-resolution mode (Sec. 3.2): positions enumerate the grid padded at the end of H and W to multiples of s*s;
    // H_real rows of every H_pad are real, and columns below W (the real row length above) are real.
    int H_real;
    FastDiv hpad;  // division by the padded H
};

__host__ __device__ inline uint32_t src_token(const GridMap& g, uint32_t p, uint32_t q, uint32_t j) {
    const uint32_t r = g.ws.div(j);
    const uint32_t ws = j - r * g.ws.d;
    const uint32_t row = r * g.a + g.sdiv.div(r) * g.b + p * g.cmul;
    const uint32_t w = ws * g.a + g.sdiv.div(ws) * g.b + q * g.cmul;
    return row * (uint32_t)g.W + w;
}

// Any-resolution mode: position j of class (p, q) on the padded grid -> token number in the UNPADDED tensor and whether the
// position is a real token.  g.ws divides by W_pad/s, g.hpad by H_pad; rows and columns of the padded grid come out of the
// same affine forms as in src_token().
__host__ __device__ inline uint32_t src_token_padded(const GridMap& g, uint32_t p, uint32_t q, uint32_t j, bool* real) {
    const uint32_t r = g.ws.div(j);
    const uint32_t ws = j - r * g.ws.d;
    const uint32_t row = r * g.a + g.sdiv.div(r) * g.b + p * g.cmul;  // t * H_pad + h
    const uint32_t w = ws * g.a + g.sdiv.div(ws) * g.b + q * g.cmul;
    const uint32_t t = g.hpad.div(row);
    const uint32_t h = row - t * g.hpad.d;
    *real = h < (uint32_t)g.H_real && w < (uint32_t)g.W;
    return (t * (uint32_t)g.H_real + h) * (uint32_t)g.W + w;
}

// Real rows (or columns) of every class along one axis in the any-resolution mode: entry 0 for the classes under `at`, 1 for class
// `at`, 2 for the others.  Three values serve every class: in the token-wise pattern the first n % s classes have one row more than
// the others; in the group-wise one the last, incomplete run of s*s rows gives s rows to some classes, the rest to one, none to others.
struct ClassAxis {
    uint32_t at;
    uint32_t n[3], mul[3];  // rows and FastDiv multiplier
    __host__ __device__ inline FastDiv of(uint32_t p) const {
        FastDiv f;
        f.d = p < at ? n[0] : p == at ? n[1] : n[2];
        f.mul = p < at ? mul[0] : p == at ? mul[1] : mul[2];
        // Formed here: kept in the arguments and selected like the others it makes the dK+dV launch (head_dim 128) spill 22 values
        // instead of 11, and the whole training step at 720P takes 115.7 ms instead of 111.2.
        f.one = f.d <= 1u ? 1u : 0u;
        return f;
    }
};

// What the kernels of the any-resolution mode need beside the GridMap; formed on the host and an argument of these kernels only, not a
// part of the map that every launch carries (a small 8-bit any-resolution call of four launches: 80.7 us with it there, 80.2).
struct PadMap {
    FastDiv hs;        // division by the padded H / s, the rows of a class on the padded grid
    ClassAxis hc, wc;  // real rows and columns of the classes
};
struct NoPadMap {};
template <bool PAD>
struct PadArgOf { typedef NoPadMap type; };
template <>
struct PadArgOf<true> { typedef PadMap type; };
template <bool PAD>
using PadArg = typename PadArgOf<PAD>::type;

// Any-resolution mode without the padding.  The padding sits at the end of H and W, so the real positions of a class are a prefix
// along either axis (both maps are monotone in hs and ws): a (T, hr, wr) grid of its own.  The attention kernels walk that grid,
// "dense" positions 0 .. n-1 with no padding among them, so that nothing is computed and masked away.
struct ClassMap {
    uint32_t n;  // real tokens of the class (0 if the unpadded grid has none)
    FastDiv w;   // division by the real columns of the class
    FastDiv h;   // division by the real rows of the class
    FastDiv hs;  // division by its rows on the padded grid
};

// Selected from values that the host forms: extents and multipliers formed in the kernel put six integer divisions in a row in front of
// every workgroup's first load (32 units of 10 tokens at head_dim 64, us a launch: 4.30 -> 4.20, in workgroups of 256 queries 4.91 -> 4.55).
__host__ __device__ inline ClassMap make_class_map(const GridMap& g, const NoPadMap&, uint32_t, uint32_t) {
    return {(uint32_t)g.n_sub, {}, {}, {}};
}
__host__ __device__ inline ClassMap make_class_map(const GridMap& g, const PadMap& m, uint32_t p, uint32_t q) {
    ClassMap c;
    c.w = m.wc.of(q);
    c.h = m.hc.of(p);
    c.n = (uint32_t)g.T * c.h.d * c.w.d;
    c.hs = m.hs;
    c.hs.one = c.hs.d <= 1u ? 1u : 0u;  // formed, as in ClassAxis
    return c;
}

// token number of dense position j of class (p, q), and the position on the padded grid that it stands for
__host__ __device__ inline uint32_t src_token_real(const GridMap& g, const ClassMap& c, uint32_t p, uint32_t q, uint32_t j) {
    const uint32_t r = c.w.div(j), ws = j - r * c.w.d;
    const uint32_t t = c.h.div(r), hs = r - t * c.h.d;
    const uint32_t h = hs * g.a + g.sdiv.div(hs) * g.b + p * g.cmul;
    const uint32_t w = ws * g.a + g.sdiv.div(ws) * g.b + q * g.cmul;
    return (t * (uint32_t)g.H_real + h) * (uint32_t)g.W + w;
}
__host__ __device__ inline uint32_t padded_position(const GridMap& g, const ClassMap& c, uint32_t j) {
    const uint32_t r = c.w.div(j), ws = j - r * c.w.d;
    const uint32_t t = c.h.div(r), hs = r - t * c.h.d;
    return (t * g.sdiv.div(g.hpad.d) + hs) * g.ws.d + ws;  // (with c.hs.d the dK+dV launch of head_dim 128 spills 17 values instead of 11)
}

// Host side: the map of a grid.  `group` selects the group-wise pattern; `pad` the any-resolution mode, in which the
// subsequences are those of the grid padded at the end of H and W to the next multiples of s*s.
inline GridMap make_dense_gridmap(size_t n) {
    GridMap g;
    g.mode = MODE_DENSE;
    g.s = 1;
    g.W = 0;
    g.n_tok = (int)n;
    g.n_sub = (int)n;
    g.T = 1;
    g.a = 1;
    g.b = 0;
    g.cmul = 0;
    g.ws = make_fastdiv(0xffffffffu);  // multiplier 2: the quotient is 0 for every position below 2^31
    g.H_real = 1;
    g.hpad = make_fastdiv(1);
    g.sdiv = make_fastdiv(1);
    return g;
}

inline GridMap make_gridmap(int T, int H, int W, int s, bool group, bool pad = false) {
    const int n_tok = T * H * W;
    if (s == 1) return make_dense_gridmap((size_t)n_tok);
    const int Hp = pad ? (H + s * s - 1) / (s * s) * (s * s) : H;
    const int Wp = pad ? (W + s * s - 1) / (s * s) * (s * s) : W;
    GridMap g;
    g.mode = group ? MODE_GROUP : MODE_TOKEN;
    g.s = s;
    g.W = W;
    g.n_tok = n_tok;
    g.n_sub = T * Hp * Wp / (s * s);
    g.T = T;
    g.a = group ? 1u : (uint32_t)s;
    g.b = group ? (uint32_t)(s * s - s) : 0u;
    g.cmul = group ? (uint32_t)s : 1u;
    g.ws = make_fastdiv((uint32_t)(Wp / s));
    g.sdiv = make_fastdiv((uint32_t)s);
    g.H_real = H;
    g.hpad = make_fastdiv((uint32_t)Hp);
    return g;
}

// Real rows (columns) of every class: n real rows in all.
inline ClassAxis make_class_axis(uint32_t n, uint32_t s, bool group) {
    const uint32_t run = group ? s : 1u;  // rows of a class that lie next to each other
    const uint32_t full = n / (s * run), rest = n - full * s * run;  // whole rounds over the classes; rows of the incomplete one
    const uint32_t len[3] = {(full + 1u) * run, full * run + rest % run, full * run};
    ClassAxis a;
    a.at = rest / run;
    for (int i = 0; i < 3; i++) {
        a.n[i] = len[i];
        a.mul[i] = make_fastdiv(len[i]).mul;
    }
    return a;
}

// The second map of an any-resolution grid (g made with pad = true).
inline PadMap make_pad_map(const GridMap& g) {
    const uint32_t s = (uint32_t)g.s;
    PadMap m;
    m.hs = make_fastdiv(g.hpad.d / s);
    m.hc = make_class_axis((uint32_t)g.H_real, s, g.mode == MODE_GROUP);
    m.wc = make_class_axis((uint32_t)g.W, s, g.mode == MODE_GROUP);
    return m;
}
inline void make_pad_arg(const GridMap&, NoPadMap&) {}
inline void make_pad_arg(const GridMap& g, PadMap& m) { m = make_pad_map(g); }
inline ClassMap make_class_map(const GridMap& g, uint32_t p, uint32_t q) { return make_class_map(g, make_pad_map(g), p, q); }

// ---- row moves: every row of one layout and where it is in another
enum RowMap : int {
    TO_SPARSE = 0,  // destination: the sparse layout, source: the original one
    TO_ORIGINAL = 1,  // the inverse
    SWITCH = 2      // destination: the sparse layout of g's pattern, source: that of the other pattern
};

// ssp_G > 0 (Sparse Sequence Parallelism, Alg. 1 sparse_sequence_parallel, step 3): the sparse side is a buffer as it arrives from the
// all-to-all, [source rank][my subsequence g'][source's subsequence g][b][position]; the algorithm's axis swap to
// [source rank][g][g'][b] = "(p q b')" order is folded into the row number instead of being a pass of its own.
__host__ __device__ inline uint32_t ssp_received_sb(uint32_t sb, uint32_t B, uint32_t G) {
    const uint32_t b = B / G;                        // batch elements per subsequence
    const uint32_t pq = sb / B, bi = sb - pq * B;    // class of the source pattern; (g', batch element)
    const uint32_t r = pq / G, gs = pq - r * G, gd = bi / b, bb = bi - gd * b;
    return ((r * G + gd) * G + gs) * b + bb;
}

// Division of any 32-bit n by any run-time constant d: the high 64 bits of n * ceil(2^64 / d), exact without a condition on the sizes
// (the multiplier is off by less than 1, the quotient by less than n / 2^64 < 1 / d).  Six scalar instructions where n is the same in every lane.
struct Div32 {
    uint32_t d, lo, hi, one;  // one: d = 1, whose multiplier would be 2^64
    __host__ __device__ inline uint32_t div(uint32_t n) const {
#if defined(__HIP_DEVICE_COMPILE__)
        const uint32_t low = __umulhi(n, lo);
#else
        const uint32_t low = (uint32_t)(((uint64_t)n * lo) >> 32);
#endif
        return (uint32_t)(((uint64_t)n * hi + low) >> 32) + n * one;
    }
};
inline Div32 make_div32(uint32_t d) {
    const uint64_t m = d <= 1u ? 0u : ~0ull / d + 1u;
    return {d, (uint32_t)m, (uint32_t)(m >> 32), d <= 1u ? 1u : 0u};
}

// Which unit, and which of its tiles, workgroup `lin` of the (unit, tile) order has.  The divisions are multiplications on the scalar unit: four divisions by
// run-time constants in a row stood in front of every workgroup's first address.
struct UnitAt {
    uint32_t unit, tile;    // unit = number in the order of the units
    uint32_t bb, head;      // subsequence (p, q, b) or batch element, and head
    uint32_t p, q, b;       // class and batch element
};
struct UnitMap {
    Div32 tiles;  // tiles of a unit
    Div32 inner;  // heads; with heads slow the subsequences, so that neighbouring units belong to different classes
    Div32 B, s;
    template <bool HEADS_SLOW>
    __host__ __device__ inline UnitAt at(uint32_t lin) const {
        UnitAt u;
        u.unit = tiles.div(lin);
        u.tile = lin - u.unit * tiles.d;
        const uint32_t slow = inner.div(u.unit), fast = u.unit - slow * inner.d;
        u.bb = HEADS_SLOW ? fast : slow;
        u.head = HEADS_SLOW ? slow : fast;
        const uint32_t pq = B.div(u.bb);
        u.b = u.bb - pq * B.d;
        u.p = s.div(pq);
        u.q = pq - u.p * s.d;
        return u;
    }
};
// (a dense map has s = 1, so that p = q = 0)
template <bool HEADS_SLOW>
inline UnitMap make_unit_map(const GridMap& g, uint32_t tiles, uint32_t B, uint32_t heads) {
    const uint32_t s = (uint32_t)g.s;
    return {make_div32(tiles), make_div32(HEADS_SLOW ? B * s * s : heads), make_div32(B), make_div32(s)};
}

// A kernel's arguments are asked for at once and waited for once: left to itself the compiler reads them where they are needed, and three or four loads from
// memory, one waiting for the other, stand in front of a workgroup's first address (35 units of 225 tokens at head_dim 64: 6.39 us so, 6.02 at once).
#define SKIPARSE_ARG_DIV32(x) "s"((x).d), "s"((x).lo), "s"((x).hi), "s"((x).one)
#define SKIPARSE_ARG_UNITS(u) SKIPARSE_ARG_DIV32((u).tiles), SKIPARSE_ARG_DIV32((u).inner), SKIPARSE_ARG_DIV32((u).B), SKIPARSE_ARG_DIV32((u).s)
#define SKIPARSE_ARG_GRID(g) "s"((g).W), "s"((g).n_tok), "s"((g).n_sub), "s"((g).a), "s"((g).b), "s"((g).cmul), "s"((g).ws.d), "s"((g).ws.mul), "s"((g).ws.one), "s"((g).sdiv.mul), "s"((g).sdiv.one)

// What the row numbers of both sides are made of, for destination rows of one RowMap.
struct RowArgs {
    Div32 n_row;    // rows of a subsequence (destination sparse) or of a batch element (destination original)
    Div32 row_len;  // W / s (destination sparse) or W
    Div32 B, s;
    uint32_t W, Ws, n_tok, n_sub;
    int mode;
};

// Algorithm 1's index maps along one axis.  x = t*H + h or w (H and W are multiples of s, and of s*s for the group-wise pattern, so t*H + h
// splits like h); (cls, pos) = the class and the place inside it.
__host__ __device__ inline void split_axis(bool group, const Div32& s, uint32_t x, uint32_t& cls, uint32_t& pos) {
    const uint32_t a = s.div(x), m = x - a * s.d;
    if (!group) {
        cls = m;
        pos = a;
        return;
    }
    const uint32_t a2 = s.div(a);
    cls = a - a2 * s.d;
    pos = a2 * s.d + m;
}
__host__ __device__ inline uint32_t join_axis(bool group, const Div32& s, uint32_t cls, uint32_t pos) {
    if (!group) return pos * s.d + cls;
    const uint32_t a = s.div(pos);
    return (a * s.d + cls) * s.d + (pos - a * s.d);
}

// row number in the source of destination row `row`
template <int MAP>
__host__ __device__ inline uint32_t source_row(const RowArgs& g, uint32_t row, uint32_t ssp_G) {
    if (g.mode == MODE_DENSE) return row;
    const bool group = g.mode == MODE_GROUP;
    const uint32_t o = g.n_row.div(row), j = row - o * g.n_row.d;  // outer number, row inside it
    const uint32_t r = g.row_len.div(j), c = j - r * g.row_len.d;
    uint32_t b = o, th = r, w = c;  // TO_ORIGINAL
    if (MAP != TO_ORIGINAL) {
        const uint32_t pq = g.B.div(o), p = g.s.div(pq);
        b = o - pq * g.B.d;
        th = join_axis(group, g.s, p, r);
        w = join_axis(group, g.s, pq - p * g.s.d, c);
        if (MAP == TO_SPARSE) return b * g.n_tok + th * g.W + w;
    }
    uint32_t p, q, pr, pc;
    split_axis(MAP == SWITCH ? !group : group, g.s, th, p, pr);
    split_axis(MAP == SWITCH ? !group : group, g.s, w, q, pc);
    uint32_t sb = (p * g.s.d + q) * g.B.d + b;
    if (MAP == TO_ORIGINAL && ssp_G) sb = ssp_received_sb(sb, g.B.d, ssp_G);
    return sb * g.n_sub + pr * g.Ws + pc;
}

// Host side: g describes the destination's pattern for TO_SPARSE and SWITCH, the source's for TO_ORIGINAL.
template <int MAP>
inline RowArgs make_row_args(const GridMap& g, uint32_t B) {
    const uint32_t W = (uint32_t)g.W, Ws = W / (uint32_t)g.s, n_tok = (uint32_t)g.n_tok, n_sub = (uint32_t)g.n_sub;
    return {make_div32(MAP == TO_ORIGINAL ? n_tok : n_sub), make_div32(MAP == TO_ORIGINAL ? W : Ws), make_div32(B), make_div32((uint32_t)g.s), W, Ws, n_tok, n_sub, g.mode};
}

}  // namespace skiparse

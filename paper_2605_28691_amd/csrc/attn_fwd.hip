// bf16 flash-attention forward for gfx950, with the Skiparse row addressing folded in.
//
// Computes, for every attention unit (a subsequence or batch element, and a head),
//     O = softmax(Q K^T * scale) V                      (Sec. 3.1: attention inside each subsequence)
// without ever forming the N x N matrix: keys are walked in blocks of 32 with a running row maximum and row sum.
//
// Mapping onto the hardware
//   * One workgroup = 4 or 8 wavefronts in one or two key groups; a wavefront owns 32 query rows, the wavefronts of a group walk the same keys
//     and share every K/V tile that is brought into LDS.  The shape for large problems is 8 wavefronts in one group: 256 queries
//     a tile halve the L2 -> LDS traffic per MFMA compared with 128 (two wavefronts per SIMD, <= 256 VGPRs per lane, 64 KiB LDS).
//     Small problems are bound by idle CUs and by the serial walk over the keys instead; they get smaller workgroups, and two
//     groups that walk half of the keys each and merge (reference, sum, O) through LDS at the end: see wg_shape.h.
//   * The products are formed transposed, S^T = K Q^T and O^T = V^T P^T, with v_mfma_f32_32x32x16_bf16.  In the
//     32x32 accumulator layout lane l holds column l%32, so every lane owns ONE query: its 16 registers per 32-key
//     block are 16 keys of that query, and the exponentiated accumulator registers, rounded to bf16, ARE the B operand
//     of the second product -- the probabilities never leave registers.  The key order inside a 16-key MFMA step is
//     whatever the accumulator layout gives (keys 4h..4h+3 and 8+4h..8+4h+3 for lane half h); V^T is fetched in the
//     same order.
//   * Software pipeline over 32-key blocks: step b issues the MFMAs of  S(b+1) = K(b+1) Q^T  and  O += V(b-1)^T P(b-1)^T
//     and does the softmax arithmetic of block b on the vector ALU.  The three are independent inside a step, so the
//     matrix pipe and the vector ALU overlap within one wavefront as well as across the two on a SIMD.
//   * In the steady state the instruction order of a step is written out by hand and fixed with scheduling fences:
//     MFMAs of the two products alternate (so consecutive MFMAs never depend on each other), each followed by its share
//     of the exponentials, and every LDS fragment is read four or eight MFMAs before its use (across the two steps of a window too).
//   * Reference maximum without a per-block maximum: the exponentials are taken against the reference the row already
//     has; the common path computes no maximum at all.  The guard is the row sum: if 16 probabilities of a lane add up
//     to 2^16 or more (always on the first block, where the reference is -inf) the wavefront takes a rare path that finds
//     the true maximum, redoes the block against it and rescales l; O is rescaled at the start of the next step in a
//     block that holds only the in-place multiplies.  In a walk's first and last windows the reference is raised from a growth of 2^8 on.  Numerator and denominator always use the same reference, so the
//     result is exact up to rounding; probabilities up to 2^16 keep their relative precision in bf16, O and l are fp32.
//   * K and V tiles of 64 keys go from global memory straight into LDS (global_load_lds_dwordx4, no staging registers,
//     no LDS store instructions), double buffered, K one tile ahead of V (a window of two steps reads K tile W and V tile
//     W-1), one barrier per window; the loads of a tile are enqueued half a window before they are waited for (not earlier:
//     see the window loop).  LDS rows are packed (a direct load writes 64 consecutive 16-byte chunks) and bank conflicts are avoided by an XOR swizzle of
//     the chunk position with the row number, chosen so that both the 16-byte fragment reads of K (16 consecutive rows)
//     and the transposing reads of V^T (ds_read_b64_tr_b16, 4 consecutive rows of 64 bytes) touch every bank once; V
//     stays row-major in LDS.  (Three buffers with a two-window lead and a fence-free barrier measured slower.)
//   * Row addresses come from the Skiparse index map: in the dense mode position j is row j, in the sparse modes it is
//     the token the rearrangement (Algorithm 1) would have put at position j, so q, k, v are read and out is written in
//     the original layout and no permuted copy exists.  The rows' byte offsets are formed 8 tiles ahead, one tile (64 rows,
//     lane = row) per window by one wavefront of the group in turn, and kept in a small ring in LDS from which every lane picks up the
//     two rows it fetches: the index arithmetic costs a wavefront one evaluation of the map per 8 tiles.
//   * Workgroups are numbered so that the query tiles of one unit run on the same XCD (workgroup id mod 8 selects
//     the XCD under round-robin dispatch; every XCD owns a contiguous eighth of the (unit, tile) order) and walk K/V in
//     step: the per-XCD L2 then serves the re-reads.
#include <type_traits>

#include "kernels.h"
#include "lds_layout.h"
#include "row_io.h"

namespace skiparse {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;

#define LDS_PTR(T) __attribute__((address_space(3))) T*

constexpr int KT = 64;          // keys per staged tile (two 32-key blocks)
static_assert(GROUP_MIN_ROWS == KT, "a key group needs a tile of its own");
constexpr int ATTN_QT = 1;       // 32-query tiles per wavefront
constexpr int RING_AHEAD = 8;    // row offsets are formed this many tiles ahead, by one wavefront per window in turn
constexpr int RING = 16;         // tiles of row offsets kept in LDS: a slot is rewritten RING - RING_AHEAD windows after its last use
static_assert((RING & (RING - 1)) == 0 && RING >= RING_AHEAD + 4, "ring sizes");
// MFMA groups by which the LDS fragment reads run ahead in the steady state.  With two wavefronts a SIMD 4 cover the latency; a single one waits for reads less
// often with 8 (48 units of 390 tokens 12.35 -> 12.13 us, training step of 48 of 400 42.4 -> 41.7; calls of several rounds as before), where the registers are there.
constexpr int lds_ahead(int D, int shape) { return shape == Q256 || shape == Q256_FULL || (D == 128 && shape == Q128_SPLIT) ? 4 : 8; }
constexpr float RESCALE_LOG2 = 8.0f;  // the reference maximum is only raised when it grew by more than 2^8

// QW: wavefronts that share a tile (and fetch it together)
template <int D, int QW>
struct Tile {
    static constexpr int CH = D / 8;                     // 16-byte chunks per row
    static constexpr int RB = D * 2;                     // row bytes in LDS: rows are packed, bank conflicts are avoided by a swizzle
    static constexpr int RPI = 64 / CH;                  // rows covered by one direct-to-LDS instruction of a wavefront (64 chunks)
    static constexpr int IPW = CH / QW;                  // such instructions per wavefront and 64-row tile
    static constexpr int TILE_BYTES = KT * RB;
    static_assert(IPW >= 1 && IPW * QW == CH, "a tile is CH instructions, spread evenly over the wavefronts");
    // chunk c of row r is stored at chunk position c ^ swz(r): see lds_layout.h
    __host__ __device__ static constexpr uint32_t swz(uint32_t r) { return lds_swizzle<D>(r); }
};

// Exchange between lanes l and l^32 (the two halves of one query's keys) with v_permlane32_swap: afterwards `lo` is
// the value of the pair's lower lane and `hi` that of its upper lane, in both lanes.  The two results are copied into
// scalars before any cast: a bit-cast applied directly to an element of the returned vector reads element 0 twice.
__device__ inline void lane_pair(float x, float& lo, float& hi) {
    const unsigned a = __float_as_uint(x);
    const auto r = __builtin_amdgcn_permlane32_swap(a, a, false, false);
    const unsigned r0 = r[0], r1 = r[1];
    lo = __uint_as_float(r0);
    hi = __uint_as_float(r1);
}

// a value that is the same in every lane, moved to a scalar register
__device__ inline uint32_t uniform(uint32_t x) { return __builtin_amdgcn_readfirstlane(x); }
__device__ inline size_t uniform(size_t x) {
    return ((size_t)uniform((uint32_t)(x >> 32)) << 32) | uniform((uint32_t)x);
}

// Row of `out` for position j of subsequence sb of the input's sparse layout: the token's row in the original layout, or its
// row in the sparse layout of the other pattern (Alg. 1: tsa_to_orig / gsa_to_orig, tsa_to_gsa / gsa_to_tsa).
__device__ inline size_t scattered_row(const AttnArgs& a, uint32_t sb, uint32_t j) {
    const GridMap& gi = a.g_in;
    const uint32_t s = (uint32_t)gi.s, W = (uint32_t)gi.W, B = (uint32_t)a.out_B;
    const uint32_t pq = sb / B, b = sb - pq * B;
    const uint32_t n = src_token(gi, pq / s, pq % s, j);
    if (a.out_kind == OUT_ORIGINAL) return (size_t)b * (uint32_t)gi.n_tok + n;
    const uint32_t th = n / W, w = n - th * W;  // th = t*H + h
    uint32_t p, q, r, ws;
    if (gi.b != 0) {  // input group-wise -> output token-wise
        p = th % s;
        q = w % s;
        r = th / s;
        ws = w / s;
    } else {          // input token-wise -> output group-wise
        p = (th / s) % s;
        q = (w / s) % s;
        r = (th / (s * s)) * s + th % s;
        ws = (w / (s * s)) * s + w % s;
    }
    return ((size_t)(p * s + q) * B + b) * (uint32_t)gi.n_sub + r * (W / s) + ws;
}

// Workgroup shapes (FwdShape): NW wavefronts in KG key groups take 32 * NW / KG queries.
constexpr int fwd_waves(int shape) { return shape == Q256 || shape == Q256_FULL || shape == Q128_SPLIT ? 8 : 4; }
constexpr int fwd_groups(int shape) { return shape == Q64_SPLIT || shape == Q128_SPLIT ? 2 : 1; }
constexpr int fwd_queries(int shape) { return 32 * fwd_waves(shape) / fwd_groups(shape) * ATTN_QT; }
// Workgroups of a shape that its rule counts on a CU: the compiler is held to the registers that they leave each other (Q128 at head_dim 64: 168, of which 165
// are in use; with a few more a third of the workgroups would wait while the rule still planned for them).  Where a workgroup was told that it has a SIMD's registers
// to itself, Q64_SPLIT at head_dim 64, the accumulators went to accumulation registers and were copied: 16 units of 250 tokens 5.64 us, so 5.03, 3 of 1600 10.3 and 9.3.
constexpr int fwd_per_cu(int D, int shape) {
    const int of = shape == Q256_FULL ? Q256 : shape == Q128_FULL ? Q128 : shape;
    for (const ShapeCost& c : D == 128 ? FWD_COST_128 : FWD_COST_64)
        if (c.shape == of) return c.max_k;
    return 1;
}

// PAD selects the any-resolution mode (Sec. 3.2), where the subsequences are those of the grid padded to multiples of s*s with the
// padding masked: the kernel walks the real tokens of the class only (ClassMap), so that a masked key is one that is never met.  Only
// the log-sum-exp is laid out over the padded grid (zero at the padding).
template <int D, int SHAPE, bool PAD>
__global__ __launch_bounds__(64 * fwd_waves(SHAPE), fwd_waves(SHAPE) / 4 * fwd_per_cu(D, SHAPE)) void attn_fwd_bf16_kernel(AttnArgs a, PadArg<PAD> pad_map, UnitMap units, uint32_t total, uint32_t per_xcd) {
    constexpr int NW = fwd_waves(SHAPE), KG = fwd_groups(SHAPE);
    constexpr int QT = ATTN_QT;
    constexpr int QW = NW / KG;    // wavefronts of a key group: each owns 32 queries, all walk the same keys
    static_assert((QW & (QW - 1)) == 0 && QW * KG == NW, "key groups are of equal size");
    using TL = Tile<D, QW>;
    constexpr int KS = D / 16;     // MFMA steps along head_dim for S^T = K Q^T
    constexpr int MT = D / 32;     // 32-row blocks of O^T
    // Small calls: the prologue forms offsets for the tiles that exist only (those past the group's last tile are read but address nothing).  With the test of
    // mask_end(), which all kernels have by now, it gave 1 to 6 % of a small launch (us, 103 units of 377 tokens at head_dim 64 12.3 -> 11.8, 144 of 160..176 in
    // the any-resolution mode at head_dim 128 12.65 -> 12.3) and cost the plain kernels of head_dim 128, which go without, three or four registers: 0.3 % at 768P
    // (110.8 -> 111.1 ms) and 0.5 % of a 13.6 us layer of 390 tokens a unit, in kernels that have been allotted anew since.
    constexpr bool TRIM = PAD || D == 64;
    constexpr bool SKIP_IDLE = SHAPE != Q256_FULL && SHAPE != Q128_FULL && !(D == 128 && SHAPE == Q64_SPLIT && !PAD);  // see fwd_kernel()
    constexpr int BR = 32 * QW * QT;   // query rows per workgroup: QT tiles of 32 per wavefront
    // four separate arrays: the compiler must be able to tell that the tile being filled is not the tile being read
    __shared__ __attribute__((aligned(1024))) char kbuf0_all[KG * TL::TILE_BYTES];
    __shared__ __attribute__((aligned(1024))) char kbuf1_all[KG * TL::TILE_BYTES];
    __shared__ __attribute__((aligned(1024))) char vbuf0_all[KG * TL::TILE_BYTES];
    __shared__ __attribute__((aligned(1024))) char vbuf1_all[KG * TL::TILE_BYTES];
    __shared__ __attribute__((aligned(16))) uint32_t rowoff_all[KG][RING][KT];        // byte offsets of the rows of the next tiles

    asm volatile("" ::SKIPARSE_ARG_UNITS(units), "s"(total), "s"(per_xcd), SKIPARSE_ARG_GRID(a.g), "s"(a.q), "s"(a.k), "s"(a.v), "s"(a.out), "s"(a.heads), "s"(a.scale), "s"(a.lse), "s"(a.out_kind));
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = uniform(tid >> 6);
    const uint32_t lq = lane & 31u, h = lane >> 5;
    const uint32_t kg = KG == 1 ? 0u : wave / QW, qw = KG == 1 ? wave : wave % QW;  // key group, wavefront of the group
    char* const kbuf0 = kbuf0_all + kg * TL::TILE_BYTES;
    char* const kbuf1 = kbuf1_all + kg * TL::TILE_BYTES;
    char* const vbuf0 = vbuf0_all + kg * TL::TILE_BYTES;
    char* const vbuf1 = vbuf1_all + kg * TL::TILE_BYTES;
    uint32_t (*const rowoff)[KT] = rowoff_all[kg];

    // workgroup -> (unit, query tile): id%8 is the XCD; each XCD owns a contiguous range of the (unit, tile) order, so that the
    // tiles of a unit run on one XCD (two at a range boundary) and the load is even for any number of units
    const uint32_t xcd = blockIdx.x & 7u, idx = blockIdx.x >> 3;
    const uint32_t lin = xcd * per_xcd + idx;
    if (lin >= total) return;
    const UnitAt at_unit = units.at<PAD>(lin);  // any-resolution mode: classes differ in size, so heads are the slow index and every XCD gets its share of each
    const uint32_t qt = at_unit.tile, bb = at_unit.bb, head = at_unit.head, p = at_unit.p, q = at_unit.q, b0 = at_unit.b;
    const ClassMap cm = make_class_map(a.g, pad_map, p, q);
    const uint32_t n_seq = PAD ? uniform(cm.n) : (uint32_t)a.g.n_sub;
    float* const lse_u = a.lse + (size_t)(bb * (uint32_t)a.heads + head) * (uint32_t)a.g.n_sub;
    if (PAD) {
        if (a.lse != nullptr)
            for (uint32_t j = qt * (64u * NW) + tid; j < (uint32_t)a.g.n_sub; j += units.tiles.d * (64u * NW)) {
                bool real;
                (void)src_token_padded(a.g, p, q, j, &real);
                if (!real) lse_u[j] = 0.f;
            }
        if (qt * BR >= n_seq) return;  // the grid is sized for the largest class
    }
    auto token_at = [&](uint32_t j) __attribute__((always_inline)) -> uint32_t {
        return PAD ? src_token_real(a.g, cm, p, q, j) : src_token(a.g, p, q, j);
    };
    const size_t C = (size_t)a.heads * D;
    const size_t unit_off = uniform((size_t)b0 * (uint32_t)a.g.n_tok * C + (size_t)head * D);  // elements
    const __bf16* Qg = (const __bf16*)a.q + unit_off;
    const __bf16* Kg = (const __bf16*)a.k + unit_off;
    const __bf16* Vg = (const __bf16*)a.v + unit_off;
    __bf16* Og = (__bf16*)a.out + unit_off;

    // ---- staging: K/V tiles of 64 rows go from global memory straight into LDS (global_load_lds_dwordx4: lane l's 16 bytes
    // land at the instruction's LDS base + 16*l, so one instruction of a wavefront fills RPI whole rows).  A wavefront issues IPW
    // such instructions per tile; lane l fetches, for row l/CH of the instruction's rows, the chunk that the swizzle puts at
    // position l%CH.  The row addresses come from the index map.
    // Byte offsets of the rows relative to the unit's base (they fit 32 bits: checked on the host) come from a small ring in LDS
    // that is filled RING_AHEAD tiles ahead: in every window ONE wavefront (they take turns) forms the 64 offsets of one tile, lane =
    // row, straight from the index map, and every lane of the workgroup later picks up the offsets of the rows it fetches.  The
    // index arithmetic thus costs each wavefront one evaluation per 8 tiles instead of one per tile and fetched row.
    const uint32_t row_bytes = (uint32_t)C * 2u;
    // the key group's share of the tiles; tiles and 32-key blocks are numbered from its start below
    const uint32_t all_tiles = (n_seq + KT - 1) / KT;
    const uint32_t tile0 = KG == 1 ? 0u : kg * all_tiles / KG;
    const uint32_t n_tiles = KG == 1 ? all_tiles : (kg + 1u) * all_tiles / KG - tile0;
    auto produce = [&](uint32_t tile) __attribute__((always_inline)) {
        const uint32_t j = (tile0 + tile) * KT + lane;
        rowoff[tile % RING][lane] = token_at(j < n_seq ? j : n_seq - 1u) * row_bytes;  // rows past the end read the last valid row
    };
    uint32_t st_row[TL::IPW], st_cb[TL::IPW];
#pragma unroll
    for (int i = 0; i < TL::IPW; i++) {
        st_row[i] = (qw * TL::IPW + i) * TL::RPI + lane / TL::CH;  // row of the tile
        st_cb[i] = ((lane % TL::CH) ^ TL::swz(st_row[i])) * 16u;  // byte offset, inside the row, of the chunk this lane fetches
    }
    struct RowOffs {
        uint32_t off[TL::IPW];  // row offset + chunk offset of the lane's fetches of one tile (the same for K and V)
    };
    auto read_offs = [&](uint32_t tile) __attribute__((always_inline)) -> RowOffs {
        RowOffs o;
#pragma unroll
        for (int i = 0; i < TL::IPW; i++) o.off[i] = rowoff[tile % RING][st_row[i]] + st_cb[i];
        return o;
    };
    // enqueue the loads of one tile; they are complete (visible in LDS after the next barrier) once tile_landed() has returned
    auto issue_tile = [&](const __bf16* g, char* buf, const RowOffs& o) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < TL::IPW; i++)
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)((const char*)g + o.off[i]),
                                             (LDS_PTR(void))(buf + (qw * TL::IPW + i) * 1024u), 16, 0, 0);
    };
    auto issue_k = [&](char* buf, const RowOffs& o) __attribute__((always_inline)) { issue_tile(Kg, buf, o); };
    auto issue_v = [&](char* buf, const RowOffs& o) __attribute__((always_inline)) { issue_tile(Vg, buf, o); };
    auto tile_landed = [&]() __attribute__((always_inline)) { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); };

    // ---- what the first window needs is asked for before anything else is formed: Q, then K tile 0, whose offsets take two trips between the lanes.  (K first, 16
    // units of 16, 64 and 160 tokens at head_dim 64 take 3.18, 3.82 and 4.89 us instead of 3.09, 3.72 and 4.80.)
    // Q fragments (B operand of S^T = K Q^T): lane = query lq, 8 consecutive channels starting at 16*ks + 8*h
    const uint32_t jq = qt * BR + qw * 32u + lq;
    const bool q_valid = jq < n_seq;
    const uint32_t q_token = token_at(q_valid ? jq : n_seq - 1u);
    const bool few = n_seq - qt * BR <= FWD_DIRECT_ROWS;  // of the workgroup's rows
    RowLoad<D> q_rows;
    bf16x8 qf[QT][KS];
    if (few) {
#pragma unroll
        for (int ks = 0; ks < KS; ks++) qf[0][ks] = *(const bf16x8*)(Qg + (size_t)q_token * C + ks * 16 + 8 * h);
    } else {
        q_rows.issue(Qg, q_token, C, lane);
    }

    // ---- K tile 0: every wavefront finds its row offsets for itself (lane = row) and hands them round its lanes.  Through the ring, K waited for an evaluation of
    // the map for every tile of the ring, a barrier and an LDS read.
    auto own_offs = [&](uint32_t tile) __attribute__((always_inline)) -> RowOffs {
        const uint32_t j = (tile0 + tile) * KT + lane;
        const uint32_t mine = token_at(j < n_seq ? j : n_seq - 1u) * row_bytes;
        RowOffs o;
#pragma unroll
        for (int i = 0; i < TL::IPW; i++) o.off[i] = (uint32_t)__shfl((int)mine, (int)st_row[i]) + st_cb[i];
        return o;
    };
    RowOffs off_v = own_offs(0);  // offsets of the tile whose V is fetched next
    issue_k(kbuf0, off_v);

    // ---- running state: every lane tracks its own query (lanes l and l^32 hold the same m_ref; l_run is a partial sum)
    f32x16 oacc[QT][MT];
    f32x16 sreg[2][QT];     // S(b) lives in sreg[b & 1]
    bf16x8 preg[2][QT][2];  // P(b) lives in preg[b & 1][query tile][16-key half]
    float m_ref[QT], l_run[QT];
#pragma unroll
    for (int qi = 0; qi < QT; qi++) {
        m_ref[qi] = -INFINITY;
        l_run[qi] = 0.f;
#pragma unroll
        for (int mt = 0; mt < MT; mt++)
#pragma unroll
            for (int r = 0; r < 16; r++) oacc[qi][mt][r] = 0.f;
    }
    const float c = a.scale * 1.4426950408889634f;  // logits are kept raw; exp(x*scale) = exp2(x*c)
    // A raised reference rescales O one step late: the factor is kept here and applied at the start of the next step
    // (after PV(b-1), before PV(b)), in a block of its own that holds nothing but the in-place multiplies.
    float alpha_pending[QT];
    bool pending = false;  // wave-uniform
#pragma unroll
    for (int qi = 0; qi < QT; qi++) alpha_pending[qi] = 1.f;
    auto apply_pending = [&]() __attribute__((always_inline)) {
        if (__builtin_expect(pending, 0)) {
#pragma unroll
            for (int qi = 0; qi < QT; qi++)
#pragma unroll
                for (int mt = 0; mt < MT; mt++)
#pragma unroll
                    for (int r = 0; r < 16; r++) oacc[qi][mt][r] *= alpha_pending[qi];
            pending = false;
        }
    };

    // LDS read offsets that do not depend on the tile
    uint32_t k_rd[KS];  // K fragment of MFMA step ks: row lq (+ 32 for the second half), chunk 2*ks + h at its swizzled position
#pragma unroll
    for (int ks = 0; ks < KS; ks++) k_rd[ks] = lq * TL::RB + (((uint32_t)(2 * ks) + h) ^ TL::swz(lq)) * 16u;
    // transposing V read: a 16-lane group covers 4 keys x 16 channels; lane i of the group addresses key i/4, channels 4*(i%4)..
    const uint32_t li = lane & 15u, lgrp = (lane >> 4) & 1u;
    uint32_t v_rd[2][MT];  // [second 4-row group][channel block]: + (half*32 + m2*16)*RB
#pragma unroll
    for (int sec = 0; sec < 2; sec++)
#pragma unroll
        for (int mt = 0; mt < MT; mt++) {
            const uint32_t row = 4 * h + (li >> 2) + 8 * sec;  // adding 16*m2 + 32*half does not change the swizzle (low 4 bits)
            const uint32_t ch = (uint32_t)(mt * 4) + lgrp * 2 + ((li & 3u) >> 1);
            v_rd[sec][mt] = row * TL::RB + ((ch ^ TL::swz(row)) * 16u) + 8 * (li & 1u);
        }

    // S(block) = K(block) Q^T from K tile buffer kb, 32-key half `half`; each K fragment feeds all QT query tiles
    auto qk = [&](const char* kb, int half, f32x16 (&s)[QT]) __attribute__((always_inline)) {
        f32x16 acc[QT];
#pragma unroll
        for (int qi = 0; qi < QT; qi++)
#pragma unroll
            for (int r = 0; r < 16; r++) acc[qi][r] = 0.f;
#pragma unroll
        for (int ks = 0; ks < KS; ks++) {
            const bf16x8 kf = *(const bf16x8*)(kb + k_rd[ks] + half * 32 * TL::RB);
#pragma unroll
            for (int qi = 0; qi < QT; qi++) {
                acc[qi] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qf[qi][ks], acc[qi], 0, 0, 0);
            }
        }
#pragma unroll
        for (int qi = 0; qi < QT; qi++) s[qi] = acc[qi];
    };
    // O^T += V(block)^T P(block)^T from V tile buffer vb, 32-key half `half`
    auto pv = [&](const char* vb, int half, const bf16x8 (&pf)[QT][2]) __attribute__((always_inline)) {
#pragma unroll
        for (int m2 = 0; m2 < 2; m2++)
#pragma unroll
            for (int mt = 0; mt < MT; mt++) {
                const char* va = vb + (half * 32 + m2 * 16) * TL::RB;
                const bf16x4 v0 = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((LDS_PTR(bf16x4))(LDS_PTR(char))(va + v_rd[0][mt]));
                const bf16x4 v1 = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((LDS_PTR(bf16x4))(LDS_PTR(char))(va + v_rd[1][mt]));
                const bf16x8 vf = __builtin_shufflevector(v0, v1, 0, 1, 2, 3, 4, 5, 6, 7);
#pragma unroll
                for (int qi = 0; qi < QT; qi++)
                    oacc[qi][mt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, pf[qi][m2], oacc[qi][mt], 0, 0, 0);
            }
    };
    auto max3 = [](float x, float y, float z) __attribute__((always_inline)) { return fmaxf(fmaxf(x, y), z); };
    // exponentials of one block against the reference mc (= m_ref * c): bf16 probabilities and their fp32 sum
    auto exps = [&](const f32x16& s, float mc, bf16x8 (&pf)[2]) __attribute__((always_inline)) -> float {
        float lsum = 0.f;
#pragma unroll
        for (int g = 0; g < 2; g++) {
            bf16x8 pk;
#pragma unroll
            for (int e = 0; e < 8; e += 2) {
                const f32x2 pe = {__builtin_amdgcn_exp2f(fmaf(s[g * 8 + e], c, -mc)), __builtin_amdgcn_exp2f(fmaf(s[g * 8 + e + 1], c, -mc))};
                const bf16x2 pb = __builtin_convertvector(pe, bf16x2);
                lsum += pe[0] + pe[1];  // row sum over the fp32 probabilities (two plain adds measure faster than one bf16 dot2)
                pk[e] = pb[0];
                pk[e + 1] = pb[1];
            }
            pf[g] = pk;
        }
        return lsum;
    };
    // logits of keys past the end, where the block holds any (wave-uniform)
    auto mask_end = [&](f32x16& s, uint32_t blk) __attribute__((always_inline)) {
        const uint32_t key0 = tile0 * KT + blk * 32u;
        if (__builtin_expect(key0 + 32u > n_seq, 0)) {
#pragma unroll
            for (int r = 0; r < 16; r++) s[r] = key0 + 8 * (r >> 2) + 4 * h + (r & 3) < n_seq ? s[r] : -INFINITY;
        }
    };
    // softmax of a block outside the pipelined steps, sreg[PAR] -> preg[PAR], by the true maximum and with keys past the end masked.  Where it raises the
    // reference, O is rescaled after PV(b-1) and before PV(b).
    auto softmax = [&](auto PARC, uint32_t blk) __attribute__((always_inline)) {
        constexpr int PAR = decltype(PARC)::value;
        unsigned long long grow_mask = 0;
#pragma unroll
        for (int qi = 0; qi < QT; qi++) {
            f32x16& s = sreg[PAR][qi];
            mask_end(s, blk);
            const float mx = fmaxf(max3(max3(s[0], s[1], s[2]), max3(s[3], s[4], s[5]), max3(s[6], s[7], s[8])),
                                   max3(max3(s[9], s[10], s[11]), max3(s[12], s[13], s[14]), s[15]));
            float lo, hi;
            lane_pair(mx, lo, hi);
            const float m_new = max3(m_ref[qi], lo, hi);
            const bool grow = (m_new - m_ref[qi]) * c > RESCALE_LOG2;  // same in lanes l and l^32
            grow_mask |= __builtin_amdgcn_ballot_w64(grow);
            const float m_use = grow ? m_new : m_ref[qi];
            // 1 where the reference stays, 0 on the first block (a group's first key is always a real one)
            alpha_pending[qi] = grow ? __builtin_amdgcn_exp2f((m_ref[qi] - m_use) * c) : 1.0f;
            m_ref[qi] = m_use;
            // the reference is still -inf only if every logit so far has overflowed to -inf: take 0 instead so that they give exp2(-inf) = 0
            const float mc_use = m_use == -INFINITY ? 0.f : m_use * c;
            l_run[qi] = fmaf(l_run[qi], alpha_pending[qi], exps(s, mc_use, preg[PAR][qi]));
        }
        pending = grow_mask != 0;
    };
    // One pipeline step for block b = 2W-1 (PAR = 1) or 2W (PAR = 0) of window W: K tile W in kb, V tile W-1 in vb.
    //   QK(b+1) -> sreg[PAR^1]   softmax(b): sreg[PAR] -> preg[PAR]   PV(b-1) with preg[PAR^1]
    // The instruction order is fixed group by group with scheduling fences, and the exponentials are taken against the reference the row already has, so the common path computes no
    // maximum at all: per key only fma, exp, half a bf16 pack and an add (row sum).  The guard is the row sum itself:
    // if a lane's 16 probabilities add up to 2^16 or more (always on the first block, where the reference is -inf), the
    // wavefront takes the rare path, which finds the true maximum, redoes the block's exponentials against it and rescales
    // O and l.  Probabilities up to 2^16 are harmless: bf16 keeps their relative precision and O, l are fp32.
    // LDS fragments are read LDS_AHEAD MFMA groups ahead and every fragment feeds the MFMAs of all QT query tiles.
    // MFMA groups of a step alternate between the two products (PV, QK, PV, QK, ...: as many of each), so consecutive MFMAs never
    // depend on each other: group g is PV group g/2 when g is even and QK group g/2 when g is odd.
    constexpr int NPV = 2 * MT, NQK = KS, NG = NPV + NQK;
    constexpr int LDS_AHEAD = lds_ahead(D, SHAPE);
    static_assert(NPV == NQK, "the two products have the same number of MFMA groups");
    // LDS fragment of group g of the step with parity PAR (its PV and QK both work on the half PAR ^ 1 of their tiles)
    auto read_frag = [&](auto PARC, const char* kb, const char* vb, int g) __attribute__((always_inline)) -> bf16x8 {
        constexpr int PAR = decltype(PARC)::value;
        const int i = g / 2;
        if (g % 2 == 0) {  // fragment of PV group i: 16-key group m2 = i / MT, channel block mt = i % MT
            const char* va = vb + ((PAR ^ 1) * 32 + (i / MT) * 16) * TL::RB;
            const bf16x4 v0 = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((LDS_PTR(bf16x4))(LDS_PTR(char))(va + v_rd[0][i % MT]));
            const bf16x4 v1 = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((LDS_PTR(bf16x4))(LDS_PTR(char))(va + v_rd[1][i % MT]));
            return __builtin_shufflevector(v0, v1, 0, 1, 2, 3, 4, 5, 6, 7);
        }
        return *(const bf16x8*)(kb + k_rd[i] + (PAR ^ 1) * 32 * TL::RB);
    };
    struct Frags {
        bf16x8 f[LDS_AHEAD];  // the first fragments of a step, read before it starts
    };
    auto first_frags = [&](auto PARC, const char* kb, const char* vb) __attribute__((always_inline)) -> Frags {
        Frags p;
#pragma unroll
        for (int g = 0; g < LDS_AHEAD; g++) p.f[g] = read_frag(PARC, kb, vb, g);
        return p;
    };
    // `pre`: the step's first LDS_AHEAD fragments, already on their way.  With NEXT the step's last groups fetch, instead of
    // nothing, the first fragments of the FOLLOWING step on the same tiles (the other parity) into `nxt`, so that the LDS
    // latency is exposed once per window instead of once per step.
    auto step_manual = [&](auto PARC, auto NEXTC, bool last, const char* kb, const char* vb, const Frags& pre, Frags& nxt) __attribute__((always_inline)) {
        constexpr int PAR = decltype(PARC)::value;
        constexpr bool NEXT = decltype(NEXTC)::value;
        using PARN = std::integral_constant<int, PAR ^ 1>;
        apply_pending();
        bf16x8 fr[NG];  // every fragment has its own name; lifetimes are short, so few registers are live at a time
#pragma unroll
        for (int g = 0; g < LDS_AHEAD; g++) fr[g] = pre.f[g];
        __builtin_amdgcn_sched_barrier(0);
        f32x16 acc[QT];
        float lsum[QT], mc[QT];
        bf16x8 pk[QT][2];
#pragma unroll
        for (int qi = 0; qi < QT; qi++) {
            lsum[qi] = 0.f;
            mc[qi] = m_ref[qi] * c;
        }
#pragma unroll
        for (int g = 0; g < NG; g++) {
            if (g + LDS_AHEAD < NG) fr[g + LDS_AHEAD] = read_frag(PARC, kb, vb, g + LDS_AHEAD);
            else if (NEXT) nxt.f[g + LDS_AHEAD - NG] = read_frag(PARN{}, kb, vb, g + LDS_AHEAD - NG);
            const int i = g / 2;
#pragma unroll
            for (int qi = 0; qi < QT; qi++) {
                if (g % 2 == 0) {
                    oacc[qi][i % MT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[g], preg[PAR ^ 1][qi][i / MT], oacc[qi][i % MT], 0, 0, 0);
                } else {
                    if (i == 0)
#pragma unroll
                        for (int r = 0; r < 16; r++) acc[qi][r] = 0.f;
                    acc[qi] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[g], qf[qi][i], acc[qi], 0, 0, 0);
                }
            }
            // this group's share of the exponentials: 16 / NG pairs of keys per query tile, rounded so that all 16 are covered
#pragma unroll
            for (int qi = 0; qi < QT; qi++) {
                const f32x16& s = sreg[PAR][qi];
#pragma unroll
                for (int e = 2 * (g * 8 / NG); e < 2 * ((g + 1) * 8 / NG); e += 2) {
                    const f32x2 pe = {__builtin_amdgcn_exp2f(fmaf(s[e], c, -mc[qi])), __builtin_amdgcn_exp2f(fmaf(s[e + 1], c, -mc[qi]))};
                    const bf16x2 pb = __builtin_convertvector(pe, bf16x2);
                    lsum[qi] += pe[0] + pe[1];
                    pk[qi][e / 8][e % 8] = pb[0];
                    pk[qi][e / 8][e % 8 + 1] = pb[1];
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        unsigned long long redo = 0;
#pragma unroll
        for (int qi = 0; qi < QT; qi++) {
            sreg[PAR ^ 1][qi] = acc[qi];
            preg[PAR][qi][0] = pk[qi][0];
            preg[PAR][qi][1] = pk[qi][1];
            asm volatile("" ::"v"(preg[PAR][qi][0]), "v"(preg[PAR][qi][1]));
            redo |= __builtin_amdgcn_ballot_w64(!(lsum[qi] < (last ? 256.0f : 65536.0f)));  // also catches inf and NaN
        }
        if (__builtin_expect(redo != 0, 0)) {
#pragma unroll
            for (int qi = 0; qi < QT; qi++) {
                f32x16& s = sreg[PAR][qi];
                const float mx = fmaxf(max3(max3(s[0], s[1], s[2]), max3(s[3], s[4], s[5]), max3(s[6], s[7], s[8])),
                                       max3(max3(s[9], s[10], s[11]), max3(s[12], s[13], s[14]), s[15]));
                float lo, hi;
                lane_pair(mx, lo, hi);
                const float m_new = max3(m_ref[qi], lo, hi);
                // a walk's last keys raise it from 2^8 on, each row for itself
                const float m_use = !last || (m_new - m_ref[qi]) * c > RESCALE_LOG2 ? m_new : m_ref[qi];
                // -inf only if every logit so far has overflowed to -inf: factor 1, exponent 0
                alpha_pending[qi] = m_use == -INFINITY ? 1.0f : __builtin_amdgcn_exp2f((m_ref[qi] - m_use) * c);  // 0 on the first block
                m_ref[qi] = m_use;
                l_run[qi] = fmaf(l_run[qi], alpha_pending[qi], exps(s, m_use == -INFINITY ? 0.f : m_use * c, preg[PAR][qi]));
            }
            pending = true;
        } else {
#pragma unroll
            for (int qi = 0; qi < QT; qi++) l_run[qi] += lsum[qi];
        }
    };
    using T_ = std::true_type;
    using F_ = std::false_type;
    using P0 = std::integral_constant<int, 0>;
    using P1 = std::integral_constant<int, 1>;

    // Staging schedule.  Window W reads K tile W and V tile W-1 from LDS.  Between its two steps it enqueues the direct loads of
    // K tile W+1 (into the K buffer that window W-1 read) and of V tile W (into the V buffer that window W-1 read); they have half
    // a window to land and are waited for just before the window's closing barrier.  The row offsets of tile W+2 are picked up
    // from the ring in window W (so that the LDS read is not waited for), and tile W+RING_AHEAD's are formed by wavefront W % QW of the group.
    // ---- prologue: offsets of tiles 1..RING_AHEAD
    for (uint32_t t = 1u + qw; t <= (uint32_t)RING_AHEAD && (!TRIM || t < n_tiles); t += QW) produce(t);
    tile_landed();
    if (!few) {  // Q's fragments, through V's buffers: V tile 0 is not asked for before the barrier
        constexpr uint32_t REGION = 2 * KG * TL::TILE_BYTES >= NW * 4096 ? 4096 : 2048;
        static_assert(NW * REGION <= 2 * KG * TL::TILE_BYTES, "a region for every wavefront");
        const uint32_t at = wave * REGION;
        q_rows.template fragments<REGION / 128>(at < KG * TL::TILE_BYTES ? vbuf0_all + at : vbuf1_all + (at - KG * TL::TILE_BYTES), qf[0], lane);
    }
    __syncthreads();
    RowOffs off_k = read_offs(1);  // offsets of the tile whose K is fetched next (past the group's last tile: read, never used)

    // ---- a wavefront without a query (in a unit's last workgroup) fetches its share of the tiles, meets the others at their barriers and
    // leaves the SIMD to the other workgroups of the CU and the power to the rest of the chip.  Out of the other wavefronts' line: in it, a call
    // without any (48 units of 1536 tokens) took 1 % longer.  (The same in the backward: 2 to 3 % gained where many units end in one, 1 to 3 % lost in all small
    // calls, whose kernels then spill and hold more code.)
    if (SKIP_IDLE && __builtin_expect(qt * BR + qw * QT * 32u >= n_seq, 0)) {
        for (uint32_t W = 0; W < n_tiles; W++) {
            if (W + 1u < n_tiles) {
                issue_k((W & 1u) ? kbuf0 : kbuf1, off_k);
                if (W != 0 && qw == (W & (uint32_t)(QW - 1))) produce(W + RING_AHEAD);
            }
            issue_v((W & 1u) ? vbuf1 : vbuf0, off_v);
            off_v = off_k;
            off_k = read_offs(W + 2u);
            tile_landed();
            __syncthreads();
        }
        if constexpr (KG > 1) {  // the barriers of the merge, where the group beside it has no query either
            if (n_tiles < (all_tiles + KG - 1) / KG) __syncthreads();
            __syncthreads();
            __syncthreads();
        }
        return;
    }
    // ---- window 0: QK(0), QK(1) and the softmax of block 0
    {
        issue_v(vbuf0, off_v);
        if (n_tiles > 1) issue_k(kbuf1, off_k);
        off_v = off_k;
        off_k = read_offs(2);
        qk(kbuf0, 0, sreg[0]);
        qk(kbuf0, 1, sreg[1]);
        softmax(P0{}, 0u);
        tile_landed();
        __syncthreads();
    }
    // ---- windows 1 .. n_tiles-1.  The parity of W selects the buffers at compile time.  The last one (MAY_END: windows that can be it) has no K tile to ask for,
    // and the block that it takes the exponentials of in its second step may hold keys past the end.  (As two steps of the generic kind, which waited for V's tile
    // in front of their LDS reads, and with the softmax and PV of a last block that has no key, 48 units of 390 tokens took 12.13 us instead of 11.62.  Offsets are
    // formed for tiles past the last as well: with a test for them 48 units of 390 tokens took 11.34 us instead of 11.08, 200 of 300 21.7 instead of 21.4, and two
    // groups the same.)
    auto window = [&](auto WP, auto MAY_END, uint32_t Wn) __attribute__((always_inline)) {
        constexpr int WPAR = decltype(WP)::value;  // Wn & 1
        char* const kb = WPAR ? kbuf1 : kbuf0;           // K tile Wn
        char* const kb_fill = WPAR ? kbuf0 : kbuf1;      // K tile Wn+1
        char* const vb = WPAR ? vbuf0 : vbuf1;           // V tile Wn-1
        char* const vb_fill = WPAR ? vbuf1 : vbuf0;      // V tile Wn
        // The next tiles' loads are enqueued between the two steps, i.e. with HALF a window of slack, on purpose.  The workgroups
        // of an XCD that walk the same unit share its K/V tiles through the L2 only while they stay close together, and what keeps
        // them together is that the one in front, which misses the L2, waits for its data while the others, which hit, catch up.
        // With a whole window of slack (loads at the window's start) even the misses are hidden, the workgroups drift apart and
        // the L2 misses quadruple (measured: 2.4e8 instead of 5.7e7 per call, and 1.6 % more time); spreading the issues over the
        // MFMA groups is slower still (each issue stalls the wavefront).
        const RowOffs off_ahead = read_offs(Wn + 2u);
        if (qw == (Wn & (uint32_t)(QW - 1))) produce(Wn + RING_AHEAD);
        const Frags pre = first_frags(P1{}, kb, vb);
        Frags mid, none;
        // The last window raises the reference where a block's maximum is above it by 2^8, as the walk's last block does: the largest probability of a row that has its
        // maximum there is 1 then, and not rounded.  With the steady state's 2^16 results were 0.2 (heads normalised) to 4 % (keys that grow along the walk) further from
        // 64 bits.  The row sum says where to look: a maximum taken over each of these blocks cost 2 to 5 % of a call, this up to 1 % where a row in 64 has grown.
        const bool last = decltype(MAY_END)::value && Wn + 1u == n_tiles;
        step_manual(P1{}, T_{}, last, kb, vb, pre, mid);
        if (!last) issue_k(kb_fill, off_k);
        issue_v(vb_fill, off_v);
        if (decltype(MAY_END)::value) mask_end(sreg[0][0], 2u * Wn);
        step_manual(P0{}, F_{}, last, kb, vb, mid, none);
        off_v = off_k;
        off_k = off_ahead;
        tile_landed();
        __syncthreads();
    };
    uint32_t W = 1;
    for (; W + 1 < n_tiles; W += 2) {
        window(P1{}, F_{}, W);
        window(P0{}, T_{}, W + 1u);
    }
    if (W < n_tiles) {
        window(P1{}, T_{}, W);
        W++;
    }
    // ---- final window (W == n_tiles): the PV of the last tile's first block, then softmax and PV of its second, if it has a key.  (As two
    // ways, each with its own copy of the first PV, 400 units of 48 tokens at head_dim 64 took 4.89 us instead of 4.75, 100 of 16 at head_dim 128 4.02 instead of 3.95.)
    {
        const char* vb = (W & 1u) ? vbuf0 : vbuf1;  // V tile W-1
        apply_pending();
        pv(vb, 0, preg[0]);
        if (tile0 * KT + (2u * W - 1u) * 32u < n_seq) {
            softmax(P1{}, 2u * W - 1u);
            apply_pending();
            pv(vb, 1, preg[1]);
        }
    }

    // ---- two key groups: each takes half of the channels and adds in the other's (reference, sum, O), through the LDS of the tiles
    constexpr int MF = MT / KG;  // channel blocks that a wavefront finishes
    static_assert(KG <= 2 && QT == 1 && QW * KG <= 8, "two groups at most, a tile buffer for each pair of wavefronts");
    auto pair_buf = [&](uint32_t g) __attribute__((always_inline)) -> char* {
        return (qw == 0 ? kbuf0_all : qw == 1 ? kbuf1_all : qw == 2 ? vbuf0_all : vbuf1_all) + g * TL::TILE_BYTES;
    };
    if constexpr (KG > 1) {
        if (n_tiles < (all_tiles + KG - 1) / KG) __syncthreads();  // a group with one tile less has passed one barrier less
        __syncthreads();                                           // every tile has been read
        __shared__ float part_ml[KG][QW][2][64];
        static_assert(MF * 4 * 1024 <= TL::TILE_BYTES && QW <= 4, "half of a wavefront's accumulators takes a group's half of a tile buffer");
        auto leave = [&](const f32x16* x) __attribute__((always_inline)) {
            char* const dst = pair_buf(kg) + lane * 16u;
#pragma unroll
            for (int m = 0; m < MF; m++)
#pragma unroll
                for (int g = 0; g < 4; g++) *(f32x4*)(dst + (m * 4 + g) * 1024) = f32x4{x[m][4 * g], x[m][4 * g + 1], x[m][4 * g + 2], x[m][4 * g + 3]};
        };
        if (kg == 0) leave(oacc[0] + MT - MF);
        else leave(oacc[0]);
        part_ml[kg][qw][0][lane] = m_ref[0];
        part_ml[kg][qw][1][lane] = l_run[0];
        __syncthreads();
        const float mo = part_ml[kg ^ 1u][qw][0][lane], lo = part_ml[kg ^ 1u][qw][1][lane];
        const float m_new = fmaxf(m_ref[0], mo);
        const float w0 = m_ref[0] == m_new ? 1.0f : __builtin_amdgcn_exp2f((m_ref[0] - m_new) * c);
        const float w1 = mo == m_new ? 1.0f : __builtin_amdgcn_exp2f((mo - m_new) * c);
        m_ref[0] = m_new;
        l_run[0] = kg == 0 ? fmaf(l_run[0], w0, lo * w1) : fmaf(lo, w1, l_run[0] * w0);
        // rounded as if the first group finished them all: a channel's bits do not depend on which group it falls to
        auto take = [&](auto FIRSTC, f32x16* x) __attribute__((always_inline)) {
            const char* const src = pair_buf(kg ^ 1u) + lane * 16u;
#pragma unroll
            for (int m = 0; m < MF; m++)
#pragma unroll
                for (int g = 0; g < 4; g++) {
                    const f32x4 o = *(const f32x4*)(src + (m * 4 + g) * 1024);
#pragma unroll
                    for (int e = 0; e < 4; e++) x[m][g * 4 + e] = decltype(FIRSTC)::value ? fmaf(o[e], w1, x[m][g * 4 + e] * w0) : fmaf(x[m][g * 4 + e], w0, o[e] * w1);
                }
        };
        if (kg == 0) take(T_{}, oacc[0]);
        else take(F_{}, oacc[0] + MT - MF);
    }

    // ---- epilogue: O = O^T / l, rounded to bf16; lane owns query lq, register r of block mt is channel 32*mt + 8*(r/4) + 4*h + r%4
    const uint32_t jw = qt * BR + qw * 32u, stored = rows_below(jw, n_seq);
    if (stored == 0u) return;
    float llo, lhi;
    lane_pair(l_run[0], llo, lhi);
    const float inv = 1.0f / (llo + lhi);
    if (a.lse != nullptr && h == 0 && kg == 0 && q_valid)
        // log-sum-exp of the scaled logits: the reference is in raw logit units, the sum is relative to it
        lse_u[PAD ? padded_position(a.g, cm, jw + lq) : jw + lq] = m_ref[0] * a.scale + __logf(llo + lhi);
    uint32_t row = q_token;
    __bf16* dst = Og + kg * (uint32_t)(D / KG);
    if (a.out_kind != OUT_AS_INPUT) {
        // the input is a sparse layout: bb is the subsequence (p, q, b) and this lane's query sits at position jw + lq of it
        dst = (__bf16*)a.out + (size_t)head * D + kg * (uint32_t)(D / KG);
        row = (uint32_t)scattered_row(a, bb, q_valid ? jw + lq : n_seq - 1u);
    }
    if (few) {
        if (stored >> lq & 1u) {
            if (KG == 1 || kg == 0) store_own_row((const f32x16(&)[MF])*oacc[0], inv, dst, row, C, lane);
            else store_own_row((const f32x16(&)[MF])*(oacc[0] + MT - MF), inv, dst, row, C, lane);
        }
        return;
    }
    // K's buffers are free here, and of the groups' buffers the half that this wavefront has taken in
    constexpr uint32_t CHP = D / KG >= 64 ? 64 : 32, REGION = KG > 1 || 2 * TL::TILE_BYTES >= NW * 4096 ? 4096 : 2048, ROWS = REGION >= 64 * CHP ? 32 : 16;
    static_assert(KG > 1 ? REGION <= TL::TILE_BYTES : NW * REGION <= 2 * TL::TILE_BYTES, "a region for every wavefront");
    const uint32_t at = qw * REGION;
    char* region;
    if constexpr (KG > 1) region = pair_buf(kg ^ 1u);
    else region = at < TL::TILE_BYTES ? kbuf0_all + at : kbuf1_all + (at - TL::TILE_BYTES);
    uint32_t lane_out = lane;  // formed anew: what Q's loads have formed of the same lane would be kept in ten registers through the whole walk
    asm volatile("" : "+v"(lane_out));
    const RowDest<CHP> dest(row, C, stored, lane_out);
    if (KG == 1 || kg == 0) store_rows<CHP, ROWS>(region, (const f32x16(&)[MF])*oacc[0], inv, dst, dest, lane_out);
    else store_rows<CHP, ROWS>(region, (const f32x16(&)[MF])*(oacc[0] + MT - MF), inv, dst, dest, lane_out);
}

template <int D, int SHAPE, bool PAD>
static hipError_t launch_t(const AttnArgs& a, uint32_t n_units, uint32_t n_max, hipStream_t stream) {
    constexpr int NW = fwd_waves(SHAPE);
    constexpr uint32_t BR = (uint32_t)fwd_queries(SHAPE);
    const uint32_t q_tiles = (n_max + BR - 1u) / BR;
    const uint64_t total = (uint64_t)n_units * q_tiles;
    if (!fits_grid(total + 7u, 64 * NW)) return hipErrorInvalidConfiguration;
    const uint32_t per_xcd = (uint32_t)((total + 7u) / 8u);
    PadArg<PAD> pad_map;
    make_pad_arg(a.g, pad_map);
    const UnitMap units = make_unit_map<PAD>(a.g, q_tiles, (uint32_t)a.B, (uint32_t)a.heads);
    attn_fwd_bf16_kernel<D, SHAPE, PAD><<<8u * per_xcd, 64 * NW, 0, stream>>>(a, pad_map, units, (uint32_t)total, per_xcd);
    return hipGetLastError();
}

template <int D, bool PAD>
static hipError_t launch_shape(const AttnArgs& a, hipStream_t stream) {
    const uint32_t s2 = a.g.mode == MODE_DENSE ? 1u : (uint32_t)(a.g.s * a.g.s);
    const uint32_t n_units = (uint32_t)a.B * s2 * (uint32_t)a.heads;
    const UnitSizes u = unit_sizes(a.g, PAD, (uint64_t)a.B * (uint32_t)a.heads);
    switch (fwd_kernel(D, PAD, u)) {
        case Q128: return launch_t<D, Q128, PAD>(a, n_units, u.n_max, stream);
        case Q64_SPLIT: return launch_t<D, Q64_SPLIT, PAD>(a, n_units, u.n_max, stream);
        case Q128_SPLIT: return launch_t<D, Q128_SPLIT, PAD>(a, n_units, u.n_max, stream);
        // (the any-resolution mode has no FULL kernels)
        case Q128_FULL: return launch_t<D, PAD ? Q128 : Q128_FULL, PAD>(a, n_units, u.n_max, stream);
        case Q256_FULL: return launch_t<D, PAD ? Q256 : Q256_FULL, PAD>(a, n_units, u.n_max, stream);
        default: return launch_t<D, Q256, PAD>(a, n_units, u.n_max, stream);
    }
}

hipError_t launch_attn_bf16(const AttnArgs& a, hipStream_t stream) {
    // one kernel serves the token-wise, group-wise and dense index maps: the map is only evaluated when the offset ring is filled
    if (a.head_dim == 128) return a.pad ? launch_shape<128, true>(a, stream) : launch_shape<128, false>(a, stream);
    if (a.head_dim == 64) return a.pad ? launch_shape<64, true>(a, stream) : launch_shape<64, false>(a, stream);
    return hipErrorInvalidValue;
}

}  // namespace skiparse

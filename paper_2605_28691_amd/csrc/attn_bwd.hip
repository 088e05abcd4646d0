// bf16 flash-attention backward for gfx950 with the Skiparse row addressing folded in (the layer is fine-tuned, Sec. 4.1, so
// it needs gradients).  For every attention unit (a subsequence and a head), with P = softmax(scale Q K^T) recomputed from
// the forward's log-sum-exp L:
//     delta_i = sum_d dO_id O_id                      (= sum_j P_ij dP_ij; formed by the dQ launch, whose owner rows hold dO, or beforehand)
//     dP = dO V^T,  dS = P o (dP - delta 1^T)
//     dQ = scale dS K,   dK = scale dS^T Q,   dV = P^T dO
// One scheme for both kinds of gradient, the forward kernel's with the roles of the tensors exchanged: a lane OWNS one row (a query for
// dQ, a key for dK+dV) and the rows of the other side are STREAMED through LDS in tiles of 64 or 32:
//     M1^T[streamed, owner] = A1 B1^T      (dQ: K Q^T;     dK+dV: Q K^T)         A1 from LDS, B1 = owner (registers)
//     M2^T[streamed, owner] = A2 B2^T      (dQ: V dO^T;    dK+dV: dO V^T)        A2 from LDS, B2 = owner (dQ: registers, dK+dV: LDS)
//     R = elementwise(M1, M2)              (dS; in the dK+dV launch also P)       registers, rounded to bf16
//     acc^T[channel, owner] += A3^T R      (dQ: K^T dS^T;  dK: Q^T dS;  dV: dO^T P)   A3 read from LDS with the transposing read
// As in the forward kernel the 32x32 accumulator layout gives every lane one owner column, so R's registers are directly the
// B operand of the last product, and the owner's gradient rows are accumulated in registers and written once: no atomics, the
// result is deterministic.  dK and dV share one walk (S and dP are formed once for both: 7 matrix products in all against the
// 5 of the definition); their two accumulators take 128 registers at head_dim 128, so the owner's V rows are kept in LDS where two
// wavefronts share a SIMD.
// Large problems at head_dim 128 whose caller has the workspace for it are one walk instead (attn_bwd_chain.hip, five products).
//   * Other large problems whose rounds of workgroups are full take a launch of each kind in workgroups of 256 owners, the least traffic per MFMA.
//     All others take ONE launch in smaller workgroups, the dK+dV ones first: a launch of each kind leaves the chip half idle in its last
//     round, which is the only one of a small problem, and two workgroups of different kinds on a CU overlap one's elementwise arithmetic
//     with the other's MFMAs.  Few units walk the streamed rows in two groups of wavefronts, half each, that add their accumulators
//     through LDS at the end (in a fixed order, so the result stays deterministic).  The rule and what it measured: wg_shape.h.
//   * log-sum-exp and delta are per QUERY: per-lane constants in the dQ launch; in the dK+dV launch per-streamed-row values,
//     staged in LDS next to the tile as -L/scale and -delta and used as the INITIAL accumulators of M1 and M2, so that
//     P = exp2(M1 * c) and dS = P o M2 need no further arithmetic (-inf / 0 for rows that must contribute nothing).
//   * Streamed tiles go from global memory straight into LDS (global_load_lds_dwordx4), rows packed, chunk positions XOR-swizzled
//     with the row number so that a tile serves both the 16-byte fragment reads and ds_read_b64_tr_b16 without bank conflicts.
//   * Rows are addressed through the Skiparse index map (Algorithm 1) exactly as in the forward kernel, so q, k, v, dO and the
//     gradients are all in the original layout.
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

#define LDS_PTR(T) __attribute__((address_space(3))) T*

constexpr int BT64 = 64;           // streamed rows per tile, but where LDS has to hold two workgroups
static_assert(GROUP_MIN_ROWS == BT64, "a group needs a tile of its own");
constexpr float LOG2E = 1.4426950408889634f;
constexpr int BRING_AHEAD = 8;   // row offsets are formed this many groups of 64 rows ahead, by one wavefront per group in turn
constexpr int BRING = 16;          // groups of 64 row offsets kept in LDS
static_assert((BRING & (BRING - 1)) == 0 && BRING >= BRING_AHEAD + 4, "ring sizes");

// LDS of a workgroup
struct BwdLds {
    char *s1buf0, *s1buf1, *s2buf0, *s2buf1;  // two streamed tensors, double buffered
    char* own2;                               // the owners' second operand, where it lives in LDS
    float *row_l, *row_d;                     // initial M1 and M2 per streamed row of both buffers (dK+dV)
    uint32_t* rowoff;                         // byte offsets of the streamed rows of the next tiles
};

// PAD: any-resolution mode (Sec. 3.2): the kernel walks the real tokens of the class only (ClassMap), so that a padding position is
// never met; log-sum-exp and delta are laid out over the padded grid.
// lin: number of the workgroup in the (unit, owner tile) order.  DELTA: the dQ part forms delta (else it is there already).
template <int D, int MODE, int NW, int KG, int BT, bool OWN2_LDS, bool DELTA, bool PAD>
__device__ __attribute__((always_inline)) inline void bwd_part(const BwdArgs& a, const PadArg<PAD>& pad_map, uint32_t lin, const UnitMap& units, const BwdLds& lds) {
    constexpr int KS = D / 16;   // MFMA steps along head_dim
    constexpr int MT = D / 32;   // 32-channel blocks of the gradient row
    constexpr int CH = D / 8;    // 16-byte chunks per row
    constexpr int RB = D * 2;    // row bytes in LDS (packed rows, swizzled chunk positions)
    constexpr int RPI = 64 / CH; // rows filled by one direct-to-LDS instruction of a wavefront
    constexpr int QW = NW / KG;  // wavefronts of a group: each owns 32 rows, all walk the same streamed rows
    constexpr int IPW = BT / RPI / QW; // such instructions per wavefront, tensor and tile
    constexpr int WGO = 32 * QW;         // owners per workgroup
    constexpr bool DKV = MODE == BWD_DKV; // dK and dV together: two accumulators
    // LDS fragments are read AH MFMA groups before their use and the order is pinned with scheduling fences, so that an MFMA
    // waits only for its own operands (left to itself the compiler issues each read right before the MFMA that needs it).
    // The dK+dV part with the owners' V in LDS has almost no registers to spare: 1 group ahead in the first two products and 2 (8 wavefronts) or 3 (4) in the
    // last two is what fits without spilling into the MFMA chains.  160 units of 960 tokens, training step, us: 375 with 1 and 2, 366 with 1 and 3 or 4, 372 with
    // 2 and 4; 48 of 400 40.3 / 39.85 / 40.1 / 40.5.  With 8 wavefronts 1 and 3 make no difference (48 units of 8190 tokens 6340 either way), and deeper variants
    // measured 2 to 14 % slower.
    constexpr int AH_A = OWN2_LDS ? 1 : 4, AH_C = OWN2_LDS ? (NW == 4 ? 3 : 2) : 4;
    constexpr int TILE_BYTES = BT * RB;
    static_assert(IPW >= 1 && IPW * QW * RPI == BT, "a tile's instructions are spread evenly over the wavefronts");
    static_assert(BT == 64 || BT == 32, "tiles of one or two blocks of 32 rows");
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t lq = lane & 31u, h = lane >> 5;
    const uint32_t kg = KG == 1 ? 0u : wave / QW, ow = KG == 1 ? wave : wave % QW;  // group, wavefront of the group
    const uint32_t gtid = tid - kg * (64u * QW);
    char* const s1buf0 = lds.s1buf0;
    char* const s1buf1 = lds.s1buf1;
    char* const s2buf0 = lds.s2buf0;
    char* const s2buf1 = lds.s2buf1;
    char* const own2buf = lds.own2;
    const uint32_t grp = kg * (uint32_t)TILE_BYTES;  // the group's half of every tile buffer: a part of the lanes' read offsets, so that it costs no register
    float (*const row_l)[BT] = (float (*)[BT])lds.row_l + kg * 2u;
    float (*const row_d)[BT] = (float (*)[BT])lds.row_d + kg * 2u;
    uint32_t* const rowoff = lds.rowoff + kg * (BRING * 64u);
    const UnitAt at_unit = units.at<PAD>(lin);  // any-resolution mode: classes differ in size, so heads are the slow index and every XCD gets its share of each
    const uint32_t ot = at_unit.tile, bb = at_unit.bb, head = at_unit.head, p = at_unit.p, q = at_unit.q, b0 = at_unit.b;
    const ClassMap cm = make_class_map(a.g, pad_map, p, q);
    const uint32_t n_seq = PAD ? __builtin_amdgcn_readfirstlane(cm.n) : (uint32_t)a.g.n_sub;
    if (PAD && ot * (uint32_t)WGO >= n_seq) return;  // the grid is sized for the largest class
    const size_t C = (size_t)a.heads * D;
    const size_t unit_off = (size_t)b0 * (uint32_t)a.g.n_tok * C + (size_t)head * D;  // elements
    const size_t row_unit = (size_t)(bb * (uint32_t)a.heads + head) * (uint32_t)a.g.n_sub;
    const float* lse_u = a.lse + row_unit;
    float* delta_u = a.delta + row_unit;

    // tensors by role
    const __bf16* own1_g = (const __bf16*)(MODE == BWD_DQ ? a.q : a.k) + unit_off;
    const __bf16* own2_g = (const __bf16*)(MODE == BWD_DQ ? a.dout : a.v) + unit_off;
    const char* st1_g = (const char*)((const __bf16*)(MODE == BWD_DQ ? a.k : a.q) + unit_off);
    const char* st2_g = (const char*)((const __bf16*)(MODE == BWD_DQ ? a.v : a.dout) + unit_off);
    __bf16* grad_g = (__bf16*)(MODE == BWD_DQ ? a.dq : a.dk) + unit_off;
    __bf16* grad2_g = (__bf16*)a.dv + unit_off;  // DKV: the second gradient

    // token at position j of this unit, and where its log-sum-exp and delta are
    auto token_at = [&](uint32_t j) __attribute__((always_inline)) -> uint32_t {
        return PAD ? src_token_real(a.g, cm, p, q, j) : src_token(a.g, p, q, j);
    };
    auto value_at = [&](uint32_t j) __attribute__((always_inline)) -> uint32_t { return PAD ? padded_position(a.g, cm, j) : j; };
    const float c = a.scale * LOG2E;  // exp(x*scale - L) = exp2(x*c - L*log2e)
    const float inv_scale = 1.0f / a.scale;

    // ---- staging of streamed tiles: global memory straight into LDS (global_load_lds_dwordx4: lane l's 16 bytes land at the
    // instruction's LDS base + 16*l, one instruction fills RPI rows).  Chunk c of row r is stored at chunk position c ^ swz(r),
    // which keeps the 16-byte fragment reads (16 consecutive rows) and the transposing reads (4 consecutive rows of 64 bytes)
    // both free of bank conflicts, so a tile that is read both ways is kept once.
    auto swz = [](uint32_t r) __attribute__((always_inline)) -> uint32_t { return lds_swizzle<D>(r); };
    // The byte offsets of the streamed rows (relative to the unit's base; they fit 32 bits: checked on the host) come from a small
    // ring in LDS filled BRING_AHEAD tiles ahead: for every tile ONE wavefront (they take turns) evaluates the index map for the 64
    // rows of a tile, lane = row, and every lane later picks up the offsets of the rows it fetches.
    const uint32_t row_bytes = (uint32_t)C * 2u;
    // the group's share of the streamed tiles; tiles are numbered from its start below
    const uint32_t all_t = (n_seq + BT - 1) / BT;
    const uint32_t tile0 = KG == 1 ? 0u : kg * all_t / KG;
    const uint32_t n_t = KG == 1 ? all_t : (kg + 1u) * all_t / KG - tile0;
    auto produce = [&](uint32_t group) __attribute__((always_inline)) {
        const uint32_t j = tile0 * BT + group * 64u + lane;
        rowoff[group % BRING * 64u + lane] = token_at(j < n_seq ? j : n_seq - 1u) * row_bytes;  // rows past the end repeat the last row
    };
    uint32_t st_row[IPW], st_cb[IPW];
#pragma unroll
    for (int i = 0; i < IPW; i++) {
        st_row[i] = (ow * IPW + i) * RPI + lane / CH;
        st_cb[i] = ((lane % CH) ^ swz(st_row[i])) * 16u;
    }
    struct RowOffs {
        uint32_t off[IPW];  // row offset + chunk offset of the lane's fetches of one tile (the same for both streamed tensors)
    };
    auto read_offs = [&](uint32_t tile) __attribute__((always_inline)) -> RowOffs {
        RowOffs o;
#pragma unroll
        for (int i = 0; i < IPW; i++) o.off[i] = rowoff[tile * BT % (BRING * 64u) + st_row[i]] + st_cb[i];
        return o;
    };
    float rl = 0.f, rd = 0.f;
    auto issue_tile = [&](uint32_t t, const RowOffs& o, char* b1, char* b2) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < IPW; i++) {
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(st1_g + o.off[i]),
                                             (LDS_PTR(void))(b1 + grp + (ow * IPW + i) * 1024u), 16, 0, 0);
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(st2_g + o.off[i]),
                                             (LDS_PTR(void))(b2 + grp + (ow * IPW + i) * 1024u), 16, 0, 0);
        }
        if (DKV && gtid < BT) {
            // log-sum-exp and delta of the streamed queries.  Nothing is done with them here: multiplied at once they were waited for, and the other wavefronts waited
            // for this one at the tile's end (us of the whole backward: 48 units of 400 tokens 28.1 -> 27.4, 24 of 1000 56.0 -> 51.8, 1 of 6116 125 -> 110, 160 of 960
            // 283 -> 273, on two launches 48 of 8190 4990 -> 4840 and 160 of 20,160 99.9 -> 97.6 ms, at head_dim 64 1 of 3955 51.1 -> 42.7).
            const uint32_t jj = (tile0 + t) * BT + gtid;
            const uint32_t at = value_at(jj < n_seq ? jj : n_seq - 1u);
            rl = lse_u[at];
            rd = delta_u[at];
        }
    };
    auto store_rowvals = [&](uint32_t t, uint32_t buf) __attribute__((always_inline)) {
        if (DKV && gtid < BT) {
            // the INITIAL accumulators of the two products, so that they cost no arithmetic of their own.  Raw logit - L/scale, times c = s*c - L*log2e; -inf
            // for a row past the end, which contributes nothing (P = 0); dP - delta
            const bool ok = (tile0 + t) * BT + gtid < n_seq;
            row_l[buf][gtid] = ok ? -rl * inv_scale : -INFINITY;
            row_d[buf][gtid] = ok ? -rd : 0.f;
        }
    };
    auto tile_landed = [&]() __attribute__((always_inline)) { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); };

    // ---- tile 0 is asked for before anything else is formed: every wavefront finds its row offsets for itself (lane = row) and hands them round its lanes
    // (Not in the any-resolution mode's dK+dV launch at head_dim 128: its registers are allotted another way then, 15 spilled values instead of 11, and at 720P it
    // takes 52.1 ms instead of 50.3.)
    constexpr bool EARLY = !(PAD && D == 128 && NW == 8 && OWN2_LDS && KG == 1);
    if constexpr (EARLY) {
        const uint32_t j = tile0 * BT + lane;
        const uint32_t mine = token_at(j < n_seq ? j : n_seq - 1u) * row_bytes;
        RowOffs o;
#pragma unroll
        for (int i = 0; i < IPW; i++) o.off[i] = (uint32_t)__shfl((int)mine, (int)st_row[i]) + st_cb[i];
        issue_tile(0, o, s1buf0, s2buf0);
    }

    // ---- owner row: operands in registers (B operands: lane = owner lq, 8 consecutive channels starting at 16*ks + 8*h)
    const uint32_t jo = ot * (uint32_t)WGO + ow * 32u + lq;
    const uint32_t jo_c = jo < n_seq ? jo : n_seq - 1u;  // an owner past the end reads the last row and stores nothing
    const uint32_t own_tok = token_at(jo_c);
    const size_t own_off = (size_t)own_tok * C;
    bf16x8 own1[KS], own2[OWN2_LDS ? 1 : KS];
#pragma unroll
    for (int ks = 0; ks < KS; ks++) {
        own1[ks] = *(const bf16x8*)(own1_g + own_off + ks * 16 + 8 * h);
        if (!OWN2_LDS) own2[OWN2_LDS ? 0 : ks] = *(const bf16x8*)(own2_g + own_off + ks * 16 + 8 * h);
    }
    float own_l = 0.f, own_d = 0.f;  // dQ: the owner is a query
    if (MODE == BWD_DQ && !DELTA) {
        const uint32_t at = value_at(jo_c);
        own_d = delta_u[at];
        own_l = lse_u[at] * LOG2E;
    }
    if (MODE == BWD_DQ && DELTA) {
        // delta of the row: its dO is here, O is read for nothing else.  Kept for the dK+dV launch, which streams the queries.
        const __bf16* o_g = (const __bf16*)a.out + unit_off + own_off;
        float sum = 0.f;
#pragma unroll
        for (int ks = 0; ks < KS; ks++) {
            const bf16x8 of = *(const bf16x8*)(o_g + ks * 16 + 8 * h);
#pragma unroll
            for (int e = 0; e < 8; e++) sum = fmaf((float)of[e], (float)own2[OWN2_LDS ? 0 : ks][e], sum);
        }
        const uint32_t at = value_at(jo_c);
        own_d = sum + __shfl_xor(sum, 32);
        own_l = lse_u[at] * LOG2E;
        if (jo < n_seq && h == 0 && kg == 0) delta_u[at] = own_d;
    }

    f32x16 acc[MT], acc2[DKV ? MT : 1];  // acc2: dV in the DKV launch
#pragma unroll
    for (int mt = 0; mt < MT; mt++)
#pragma unroll
        for (int r = 0; r < 16; r++) {
            acc[mt][r] = 0.f;
            if (DKV) acc2[mt][r] = 0.f;
        }

    // fragment of MFMA step ks: row lq (+ 32*blk), chunk 2*ks + h at its swizzled position.  The position of step ks is that of
    // step 0 with ks*32 XORed in (the row part lies above the chunk bits), so one register and an XOR per read can replace the
    // table; the dK+dV launch, the tightest on registers, does that.
    constexpr bool ADDR_TABLE = !DKV;
    const uint32_t a_rd0 = grp + lq * RB + ((h ^ swz(lq)) * 16u);
    uint32_t a_rd_tab[ADDR_TABLE ? KS : 1];
    if (ADDR_TABLE) {
#pragma unroll
        for (int ks = 0; ks < KS; ks++) a_rd_tab[ks] = a_rd0 ^ (uint32_t)(ks * 32);
    }
    auto a_rd = [&](int ks) __attribute__((always_inline)) -> uint32_t { return ADDR_TABLE ? a_rd_tab[ks] : (a_rd0 ^ (uint32_t)(ks * 32)); };
    // transposing read: a 16-lane group covers 4 rows x 16 channels; lane i of the group addresses row i/4, channels 4*(i%4)..
    const uint32_t li = lane & 15u, lgrp = (lane >> 4) & 1u;
    uint32_t t_rd[2][MT];  // [second 4-row group][channel block]: + (blk*32 + g2*16)*RB
#pragma unroll
    for (int sec = 0; sec < 2; sec++)
#pragma unroll
        for (int mt = 0; mt < MT; mt++) {
            const uint32_t row = 4 * h + (li >> 2) + 8 * sec;  // adding 16*g2 + 32*blk does not change the swizzle (low 4 bits)
            const uint32_t ch = (uint32_t)(mt * 4) + lgrp * 2 + ((li & 3u) >> 1);
            t_rd[sec][mt] = grp + row * RB + ((ch ^ swz(row)) * 16u) + 8 * (li & 1u);
        }

    if (OWN2_LDS) {
        // the wavefront's owner rows of V go straight into LDS (one instruction fills RPI rows; same swizzle as the tiles, so
        // the fragment of MFMA step ks sits at a_rd(ks) of a 32-row block); waited for with tile 0
#pragma unroll
        for (int i0 = 0; i0 < 32 / RPI; i0 += KG) {
            const uint32_t i = (uint32_t)i0 + kg, r = i * RPI + lane / CH;  // row of the wavefront's block; the groups have the same owners
            const uint32_t j = ot * (uint32_t)WGO + ow * 32u + r;
            const uint32_t off = token_at(j < n_seq ? j : n_seq - 1u) * row_bytes + (((lane % CH) ^ swz(r)) * 16u);
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)((const char*)own2_g + off),
                                             (LDS_PTR(void))(own2buf + ow * 32u * RB + i * 1024u), 16, 0, 0);
        }
    }
    const char* const own2_lds = own2buf + (OWN2_LDS ? ow * 32u * RB : 0u) - grp;  // read at a_rd()
    for (uint32_t t = EARLY && BT == 64 ? 1u + ow : ow; t < (uint32_t)BRING_AHEAD; t += QW) produce(t);
    if constexpr (!EARLY) {
        __syncthreads();
        issue_tile(0, read_offs(0), s1buf0, s2buf0);
    }
    store_rowvals(0, 0);
    tile_landed();
    __syncthreads();
    RowOffs off_next = read_offs(1);
    // one tile: enqueue the loads of the next tile into the other buffers, compute on this one, wait, barrier.  The parity of
    // the tile (which buffers) is a compile-time constant.  Tile t also forms the row offsets of tile t + BRING_AHEAD (written
    // here, first read in tile t + BRING_AHEAD - 2; the slot's previous tenant, tile t + BRING_AHEAD - BRING, was last read in tile
    // t + BRING_AHEAD - BRING - 1: barriers lie between in both directions).
    // The last tile is the only one that may hold streamed rows past the end; in the dQ launch they are masked.  PEEL: the last tiles
    // are code of their own, so that the loop has neither the selects nor the test for a next tile (head_dim 64 -5..-9 %, the others
    // -1..-3 %); the kernels at the register limit (head_dim 128 with two wavefronts per SIMD) spill when the copies are laid out in a
    // row (414 values in the dK+dV launch, +20 %) and keep the test.
    constexpr bool PEEL = BT == 64 && !(D == 128 && (NW == 8 || (KG == 1 && MODE == BWD_DQ)));
    auto do_tile = [&](auto PARC, auto LASTC, uint32_t t) __attribute__((always_inline)) {
        const bool more = PEEL ? !decltype(LASTC)::value : t + 1 < n_t;
        const bool tail = MODE == BWD_DQ && !more && n_seq % BT != 0 && kg == KG - 1;
        constexpr int PARITY = decltype(PARC)::value;  // t & 1
        const char* t1 = PARITY ? s1buf1 : s1buf0;
        const char* t2 = PARITY ? s2buf1 : s2buf0;
        const RowOffs off_now = off_next;
        off_next = read_offs(t + 2u);  // picked up a tile early so that the LDS read is not waited for
        if (BT == 64) {
            if (ow == (t & (uint32_t)(QW - 1))) produce(t + BRING_AHEAD);
        } else if (PARITY == 0) {
            if (ow == (t / 2u & (uint32_t)(QW - 1))) produce(t / 2u + BRING_AHEAD);
        }
#pragma unroll
        for (int blk = 0; blk < BT / 32; blk++) {
            // The next tile's loads are enqueued halfway through this one on purpose: with a whole tile of slack even L2 misses are
            // hidden, the workgroups that walk the same unit drift apart and stop sharing its tiles through the L2.
            if (blk == BT / 32 - 1 && more) issue_tile(t + 1, off_now, PARITY ? s1buf0 : s1buf1, PARITY ? s2buf0 : s2buf1);
            // register r of a block is streamed row 8*(r/4) + 4*h + r%4; the per-row values start the accumulators
            f32x16 m1, m2;
#pragma unroll
            for (int g = 0; g < 4; g++) {
                f32x4 i1 = {0.f, 0.f, 0.f, 0.f}, i2 = {0.f, 0.f, 0.f, 0.f};
                if (DKV) i1 = *(const f32x4*)&row_l[PARITY][blk * 32 + 8 * g + 4 * h];
                if (DKV) i2 = *(const f32x4*)&row_d[PARITY][blk * 32 + 8 * g + 4 * h];
#pragma unroll
                for (int e = 0; e < 4; e++) {
                    m1[4 * g + e] = i1[e];
                    m2[4 * g + e] = i2[e];
                }
            }
            // M1 and M2: their MFMA steps alternate (two independent accumulators)
            constexpr int NA = 2 * KS;
            auto frag_a = [&](int g) __attribute__((always_inline)) -> bf16x8 {
                return *(const bf16x8*)((g % 2 == 0 ? t1 : t2) + a_rd(g / 2) + blk * 32 * RB);
            };
            bf16x8 fa[NA], oa[OWN2_LDS ? KS : 1];
            auto read_a = [&](int g) __attribute__((always_inline)) {
                fa[g] = frag_a(g);
                if (OWN2_LDS && g % 2 == 1) oa[OWN2_LDS ? g / 2 : 0] = *(const bf16x8*)(own2_lds + a_rd(g / 2));
            };
#pragma unroll
            for (int g = 0; g < AH_A; g++) read_a(g);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int g = 0; g < NA; g++) {
                if (g + AH_A < NA) read_a(g + AH_A);
                if (g % 2 == 0) m1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[g], own1[g / 2], m1, 0, 0, 0);
                else m2 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[g], OWN2_LDS ? oa[OWN2_LDS ? g / 2 : 0] : own2[OWN2_LDS ? 0 : g / 2], m2, 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
            // the last product's first fragments are fetched now, under the elementwise arithmetic
            constexpr int NC = (DKV ? 4 : 2) * MT;  // DKV: dK and dV groups alternate
            auto frag_c = [&](int cidx) __attribute__((always_inline)) -> bf16x8 {
                const int pair = DKV ? cidx / 2 : cidx, g2 = pair / MT, mt = pair % MT;
                const char* ta = ((DKV && cidx % 2 == 1) ? t2 : t1) + (blk * 32 + g2 * 16) * RB;  // dV reads the dO tile, dQ and dK the first tensor
                // the offset of channel block mt is that of block 0 with mt * 64 XORed in (the swizzle moves only bits 4-7, and the
                // block number enters through bits 6-7): the dK+dV launch keeps two registers instead of the table
                const uint32_t o0 = ADDR_TABLE ? t_rd[0][mt] : (t_rd[0][0] ^ (uint32_t)(mt * 64));
                const uint32_t o1 = ADDR_TABLE ? t_rd[1][mt] : (t_rd[1][0] ^ (uint32_t)(mt * 64));
                const bf16x4 v0 = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((LDS_PTR(bf16x4))(LDS_PTR(char))(ta + o0));
                const bf16x4 v1 = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((LDS_PTR(bf16x4))(LDS_PTR(char))(ta + o1));
                return __builtin_shufflevector(v0, v1, 0, 1, 2, 3, 4, 5, 6, 7);
            };
            bf16x8 fc[NC];
#pragma unroll
            for (int cidx = 0; cidx < AH_C; cidx++) fc[cidx] = frag_c(cidx);
            __builtin_amdgcn_sched_barrier(0);
            bf16x8 rf[2], rp[DKV ? 2 : 1];  // rp: P itself in the DKV launch (rf holds dS there)
#pragma unroll
            for (int g2 = 0; g2 < 2; g2++) {
                bf16x8 pk, pp;
#pragma unroll
                for (int e = 0; e < 8; e += 2) {
                    f32x2 val, prob;
#pragma unroll
                    for (int u = 0; u < 2; u++) {
                        const int r = g2 * 8 + e + u;
                        float pr = MODE == BWD_DQ ? __builtin_amdgcn_exp2f(fmaf(m1[r], c, -own_l)) : __builtin_amdgcn_exp2f(m1[r] * c);
                        if (tail) {
                            const uint32_t row = (tile0 + t) * BT + blk * 32 + 8 * (r >> 2) + 4 * h + (r & 3);
                            pr = row < n_seq ? pr : 0.f;
                        }
                        val[u] = MODE == BWD_DQ ? pr * (m2[r] - own_d) : pr * m2[r];
                        prob[u] = pr;
                    }
                    const bf16x2 vb = __builtin_convertvector(val, bf16x2);
                    pk[e] = vb[0];
                    pk[e + 1] = vb[1];
                    if (DKV) {
                        const bf16x2 pb = __builtin_convertvector(prob, bf16x2);
                        pp[e] = pb[0];
                        pp[e + 1] = pb[1];
                    }
                }
                rf[g2] = pk;
                if (DKV) rp[g2] = pp;
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int cidx = 0; cidx < NC; cidx++) {
                if (cidx + AH_C < NC) fc[cidx + AH_C] = frag_c(cidx + AH_C);
                const int pair = DKV ? cidx / 2 : cidx, g2 = pair / MT, mt = pair % MT;
                if (DKV && cidx % 2 == 1) acc2[mt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fc[cidx], rp[DKV ? g2 : 0], acc2[mt], 0, 0, 0);  // dV^T += dO^T P
                else acc[mt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fc[cidx], rf[g2], acc[mt], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        if (more) store_rowvals(t + 1u, PARITY ^ 1);
        tile_landed();
        __syncthreads();
    };
    using P0 = std::integral_constant<int, 0>;
    using P1 = std::integral_constant<int, 1>;
    uint32_t t = 0;
    if constexpr (PEEL) {
        for (; t + 2 < n_t; t += 2) {
            do_tile(P0{}, std::false_type{}, t);
            do_tile(P1{}, std::false_type{}, t + 1u);
        }
        if (t + 1 < n_t) {
            do_tile(P0{}, std::false_type{}, t);
            do_tile(P1{}, std::true_type{}, t + 1u);
        } else if (t < n_t) {
            do_tile(P0{}, std::true_type{}, t);
        }
    } else {
        for (; t + 1 < n_t; t += 2) {
            do_tile(P0{}, std::false_type{}, t);
            do_tile(P1{}, std::false_type{}, t + 1u);
        }
        if (t < n_t) do_tile(P0{}, std::false_type{}, t);
    }

    // ---- two groups: one finishes dK and the other dV, or each half of dQ's channels, adding the other group's sums to its own, through the LDS of the tiles
    constexpr int MF = KG > 1 && !DKV ? MT / 2 : MT;  // channel blocks that a wavefront finishes
    static_assert(KG <= 2 && QW * KG <= 8, "two groups at most");
    constexpr uint32_t PART = MF * 4 * 1024;  // of a wavefront
    auto part = [&](uint32_t i) __attribute__((always_inline)) -> char* {
        const uint32_t n = i % 4u;
        return (n == 0 ? s1buf0 : n == 1 ? s1buf1 : n == 2 ? s2buf0 : s2buf1) + i / 4u * PART;
    };
    const uint32_t jw = ot * (uint32_t)WGO + ow * 32u, stored = rows_below(jw, n_seq);
    const bool few = !DELTA && n_seq - ot * (uint32_t)WGO <= BWD_DIRECT_ROWS;  // of the workgroup's rows; the launches of one kind are for long units
    if constexpr (KG > 1) {
        if (n_t < (all_t + KG - 1) / KG) __syncthreads();  // a group with one tile less has passed one barrier less
        // every tile has been read (each ends with a barrier)
        constexpr bool AT_ONCE = KG * QW <= 4 * KG * TILE_BYTES / (int)PART;  // room for both directions
        static_assert(QW <= 4 && KG * TILE_BYTES % PART == 0 && PART >= 4096, "the tile buffers hold what every wavefront of a group leaves");
        auto leave = [&](char* dst, const f32x16* x) __attribute__((always_inline)) {
#pragma unroll
            for (int m = 0; m < MF; m++)
#pragma unroll
                for (int g = 0; g < 4; g++) *(f32x4*)(dst + lane * 16u + (m * 4 + g) * 1024) = f32x4{x[m][4 * g], x[m][4 * g + 1], x[m][4 * g + 2], x[m][4 * g + 3]};
        };
        auto take = [&](const char* src, f32x16* x) __attribute__((always_inline)) {
#pragma unroll
            for (int m = 0; m < MF; m++)
#pragma unroll
                for (int g = 0; g < 4; g++) {
                    const f32x4 o = *(const f32x4*)(src + lane * 16u + (m * 4 + g) * 1024);
#pragma unroll
                    for (int e = 0; e < 4; e++) x[m][4 * g + e] += o[e];
                }
        };
        f32x16* const second = DKV ? acc2 : acc + MT - MF;  // group 1's
        // part(ow) from group 1 to group 0, part(QW + ow) (the same one, with a barrier more, where there is no room) the other way
        char *const to0 = part(ow), *const to1 = part(AT_ONCE ? QW + ow : ow);
        if (kg != 0) leave(to0, acc);
        else if (AT_ONCE) leave(to1, second);
        __syncthreads();
        if (kg == 0) take(to0, acc);
        if (!AT_ONCE) {
            __syncthreads();
            if (kg == 0) leave(to1, second);
            __syncthreads();
        }
        if (kg != 0) take(to1, second);
        if (stored == 0u) return;
        if (few) {
            if (stored >> lq & 1u) {
                if (kg == 0) store_own_row((const f32x16(&)[MF])*acc, a.scale, grad_g, own_tok, C, lane);
                else store_own_row((const f32x16(&)[MF])*second, DKV ? 1.0f : a.scale, DKV ? grad2_g : grad_g + D / 2, own_tok, C, lane);
            }
            return;
        }
        // a wavefront's region: what it has taken; without room for both that is group 1's, and group 0 has the owners' second operand instead
        static_assert(AT_ONCE || OWN2_LDS, "a region for group 0");
        constexpr int CHP = MF * 32 >= 64 ? 64 : 32;
        const RowDest<CHP> dest(own_tok, C, stored, lane);
        if (kg == 0) store_rows<CHP, 32>(AT_ONCE ? to0 : own2buf + ow * 32u * RB, (const f32x16(&)[MF])*acc, a.scale, grad_g, dest, lane);
        else store_rows<CHP, 32>(to1, (const f32x16(&)[MF])*second, DKV ? 1.0f : a.scale, DKV ? grad2_g : grad_g + D / 2, dest, lane);
        return;
    }

    // ---- epilogue: lane owns row jo; every tile has been read, 4 KiB of the buffers for each wavefront
    if (stored == 0u) return;
    if (few) {
        if (stored >> lq & 1u) {
            store_own_row(acc, a.scale, grad_g, own_tok, C, lane);
            if constexpr (DKV) store_own_row(acc2, 1.0f, grad2_g, own_tok, C, lane);
        }
        return;
    }
    constexpr uint32_t PER_BUF = TILE_BYTES / 4096;
    static_assert(KG > 1 || NW <= 4 * (int)PER_BUF, "a region of the tile buffers for every wavefront");
    const uint32_t in = ow / PER_BUF;
    char* const region = (in == 0 ? s1buf0 : in == 1 ? s1buf1 : in == 2 ? s2buf0 : s2buf1) + ow % PER_BUF * 4096u;
    const RowDest<64> dest(own_tok, C, stored, lane);
    store_rows<64, 32>(region, acc, a.scale, grad_g, dest, lane);
    if constexpr (DKV) store_rows<64, 32>(region, acc2, 1.0f, grad2_g, dest, lane);
}

// A launch of one kind of owner.
template <int D, int MODE, int NW, bool PAD>
__global__ __launch_bounds__(64 * NW, (NW == 4 ? 2 : 1)) void attn_bwd_kernel(BwdArgs a, PadArg<PAD> pad_map, UnitMap units, uint32_t total, uint32_t per_xcd) {
    constexpr bool OWN2_LDS = MODE == BWD_DKV;
    constexpr int TILE = BT64 * D * 2;
    // separate arrays so that the compiler can tell the tile being filled from the one being read
    __shared__ __attribute__((aligned(1024))) char s1buf0[TILE], s1buf1[TILE], s2buf0[TILE], s2buf1[TILE];
    __shared__ __attribute__((aligned(1024))) char own2[OWN2_LDS ? 32 * NW * D * 2 : 16];  // V rows of the owners, swizzled like a tile
    __shared__ __attribute__((aligned(16))) float row_l[2 * BT64], row_d[2 * BT64];
    __shared__ __attribute__((aligned(16))) uint32_t rowoff[BRING * 64];
    asm volatile("" ::SKIPARSE_ARG_UNITS(units), "s"(total), "s"(per_xcd), SKIPARSE_ARG_GRID(a.g), "s"(a.q), "s"(a.k), "s"(a.v), "s"(a.out), "s"(a.dout), "s"(a.lse), "s"(a.delta), "s"(a.dq), "s"(a.dk), "s"(a.dv), "s"(a.heads), "s"(a.scale));
    const uint32_t lin = (blockIdx.x & 7u) * per_xcd + (blockIdx.x >> 3);  // each XCD owns a contiguous range of the (unit, owner tile) order
    if (lin >= total) return;
    bwd_part<D, MODE, NW, 1, BT64, OWN2_LDS, true, PAD>(a, pad_map, lin, units, {s1buf0, s1buf1, s2buf0, s2buf1, own2, row_l, row_d, rowoff});
}

// Both kinds in one launch.  At head_dim 128 with the owners' V in LDS, tiles of 32 rows leave room for two B128 workgroups on a CU (70 KiB each) and
// for the two groups of B128_SPLIT; each kind fits 256 registers without a spill (4 or 5 values in B128_SPLIT).  48 units of 400 tokens: 30 us with the
// launch that forms delta, 160 of 960: 290 (650 TFLOP/s on the definition's five products); 35 and 312 when it was compared with a launch of each kind, 43 and 344.
constexpr int both_waves(int shape) { return shape == B128_SPLIT ? 8 : 4; }
constexpr int both_groups(int shape) { return shape == B128 ? 1 : 2; }
template <int D, int SHAPE, bool PAD>
__global__ __launch_bounds__(64 * both_waves(SHAPE), (SHAPE == B128 || (SHAPE == B64_SPLIT && D == 64) ? 2 : 1)) void attn_bwd_both_kernel(BwdArgs a, PadArg<PAD> pad_map, UnitMap units, uint32_t total, uint32_t per_xcd) {
    constexpr int NW = both_waves(SHAPE), KG = both_groups(SHAPE);
    constexpr bool OWN2_LDS = D == 128 && SHAPE != B64_SPLIT;
    constexpr int BT = OWN2_LDS ? 32 : BT64, TILE = BT * D * 2;
    __shared__ __attribute__((aligned(1024))) char s1buf0[KG * TILE], s1buf1[KG * TILE], s2buf0[KG * TILE], s2buf1[KG * TILE];
    __shared__ __attribute__((aligned(1024))) char own2[OWN2_LDS ? 32 * NW / KG * D * 2 : 16];
    __shared__ __attribute__((aligned(16))) float row_l[KG * 2 * BT], row_d[KG * 2 * BT];
    __shared__ __attribute__((aligned(16))) uint32_t rowoff[KG * BRING * 64];
    asm volatile("" ::SKIPARSE_ARG_UNITS(units), "s"(total), "s"(per_xcd), SKIPARSE_ARG_GRID(a.g), "s"(a.q), "s"(a.k), "s"(a.v), "s"(a.out), "s"(a.dout), "s"(a.lse), "s"(a.delta), "s"(a.dq), "s"(a.dk), "s"(a.dv), "s"(a.heads), "s"(a.scale));
    const bool dkv = blockIdx.y == 0;  // the longer workgroups first: what is left over at the end is short
    const uint32_t lin = (blockIdx.x & 7u) * per_xcd + (blockIdx.x >> 3);
    if (lin >= total) return;
    const BwdLds lds = {s1buf0, s1buf1, s2buf0, s2buf1, own2, row_l, row_d, rowoff};
    if (dkv) bwd_part<D, BWD_DKV, NW, KG, BT, OWN2_LDS, false, PAD>(a, pad_map, lin, units, lds);
    else bwd_part<D, BWD_DQ, NW, KG, BT, false, false, PAD>(a, pad_map, lin, units, lds);
}

// delta = rowsum(dO o O) of every query, for the launch of both kinds.  A wavefront takes 16 rows of a unit, lane i finding row i, with all loads
// in flight at once.  HBM-bound where it is not a launch's latency: 160 units of 960 tokens at head_dim 128 take 13 us of 290.
// CHAIN: for attn_bwd_chain.hip, what its steps start their products with instead, its control words cleared, and the gradients of every block of keys marked as missing.
struct NoChain {};
template <int D, bool PAD, typename Chain>
__global__ __launch_bounds__(256) void attn_bwd_delta_kernel(BwdArgs a, PadArg<PAD> pad_map, UnitMap units, uint32_t total, Chain chain) {
    constexpr bool CHAIN = std::is_same<Chain, BwdChain>::value;
    constexpr int CH = D / 8, RPI = 64 / CH, N = 16 / RPI;  // lanes a row, rows an instruction, instructions
    asm volatile("" ::SKIPARSE_ARG_UNITS(units), "s"(total), SKIPARSE_ARG_GRID(a.g), "s"(a.out), "s"(a.dout), "s"(a.delta), "s"(a.heads));
    if constexpr (CHAIN)
        for (uint32_t i = blockIdx.x * 256u + threadIdx.x; i < chain.n_ctl(); i += gridDim.x * 256u) chain.ctl[i] = 0u;
    const uint32_t lane = threadIdx.x & 63u, id = __builtin_amdgcn_readfirstlane(blockIdx.x * 4u + (threadIdx.x >> 6));
    if (id >= total) return;
    const UnitAt at_unit = units.at<false>(id);
    const uint32_t unit = at_unit.unit, j0 = at_unit.tile * 16u, head = at_unit.head, p = at_unit.p, q = at_unit.q, b0 = at_unit.b;
    const ClassMap cm = make_class_map(a.g, pad_map, p, q);
    const uint32_t n_seq = PAD ? cm.n : (uint32_t)a.g.n_sub;
    if (j0 >= (CHAIN ? (n_seq + CHAIN_STEP - 1u) / CHAIN_STEP * CHAIN_STEP : n_seq)) return;
    const uint32_t jl = j0 + (lane & 15u), jc = jl < n_seq ? jl : n_seq - 1u;
    const uint32_t tok = PAD ? src_token_real(a.g, cm, p, q, jc) : src_token(a.g, p, q, jc), at = PAD ? padded_position(a.g, cm, jc) : jc;
    const size_t C = (size_t)a.heads * D, base = (size_t)b0 * (uint32_t)a.g.n_tok * C + (size_t)head * D + lane % CH * 8u;
    const __bf16 *o_g = (const __bf16*)a.out + base, *do_g = (const __bf16*)a.dout + base;
    bf16x8 o[N], d[N];
#pragma unroll
    for (int i = 0; i < N; i++) {
        const size_t row = (size_t)(uint32_t)__shfl((int)tok, (int)(i * RPI + lane / CH)) * C;
        o[i] = *(const bf16x8*)(o_g + row);
        d[i] = *(const bf16x8*)(do_g + row);
    }
    if constexpr (CHAIN) {
        // One value of every block of keys is no number until the walk has written the block: what it were to leave out (take_task() in attn_bwd_chain.hip) would show.
        if (lane == 0u && j0 % CHAIN_OWNERS == 0u) {
            const size_t first = base + (size_t)tok * C;
            ((__bf16*)a.dq)[first] = ((__bf16*)a.dk)[first] = ((__bf16*)a.dv)[first] = (__bf16)__builtin_nanf("");
        }
    }
    float* delta_u = a.delta + (size_t)unit * (uint32_t)a.g.n_sub;
    const float* lse_u = a.lse + (size_t)unit * (uint32_t)a.g.n_sub;
#pragma unroll
    for (int i = 0; i < N; i++) {
        float sum = 0.f;
#pragma unroll
        for (int e = 0; e < 8; e++) sum = fmaf((float)o[i][e], (float)d[i][e], sum);
#pragma unroll
        for (int off = 1; off < CH; off <<= 1) sum += __shfl_xor(sum, off);
        const uint32_t r = i * RPI + lane / CH, pos = (uint32_t)__shfl((int)at, (int)r);
        if constexpr (CHAIN) {
            if (lane % CH == 0) {
                const uint32_t j = j0 + r;
                float* const at = chain.vals + ((size_t)unit * chain.n_steps + j / CHAIN_STEP) * (2u * CHAIN_STEP) + j % CHAIN_STEP;
                at[0] = j < n_seq ? -lse_u[pos] * (1.0f / a.scale) : -INFINITY;
                at[CHAIN_STEP] = j < n_seq ? -sum : 0.f;
            }
        } else if (lane % CH == 0 && j0 + r < n_seq) {
            delta_u[pos] = sum;
        }
    }
}

template <int D, bool PAD, typename Chain>
static hipError_t launch_delta(const BwdArgs& a, uint32_t n_units, uint32_t n_rows, const Chain& chain, hipStream_t stream) {
    const uint32_t d_tiles = (n_rows + 15u) / 16u;
    const uint64_t waves = (uint64_t)n_units * d_tiles;
    if (!fits_grid((waves + 3u) / 4u, 256u)) return hipErrorInvalidConfiguration;
    PadArg<PAD> pad_map;
    make_pad_arg(a.g, pad_map);
    attn_bwd_delta_kernel<D, PAD, Chain><<<(uint32_t)((waves + 3u) / 4u), 256, 0, stream>>>(a, pad_map, make_unit_map<false>(a.g, d_tiles, (uint32_t)a.B, (uint32_t)a.heads), (uint32_t)waves, chain);
    return hipGetLastError();
}

template <int D, int SHAPE, bool PAD>
static hipError_t launch_both(const BwdArgs& a, uint32_t n_units, uint32_t n_max, hipStream_t stream) {
    constexpr uint32_t NW = both_waves(SHAPE), WGO = 32u * NW / both_groups(SHAPE);
    const uint32_t o_tiles = (n_max + WGO - 1u) / WGO;
    const uint64_t total = (uint64_t)n_units * o_tiles;
    if (!fits_grid(total + 7u, 64u * NW)) return hipErrorInvalidConfiguration;
    const uint32_t per_xcd = (uint32_t)((total + 7u) / 8u);
    PadArg<PAD> pad_map;
    make_pad_arg(a.g, pad_map);
    const hipError_t e = launch_delta<D, PAD>(a, n_units, n_max, NoChain{}, stream);
    if (e != hipSuccess) return e;
    // a dimension of the grid for each kind: together they could fill one
    attn_bwd_both_kernel<D, SHAPE, PAD><<<dim3(8u * per_xcd, 2u), 64u * NW, 0, stream>>>(a, pad_map, make_unit_map<PAD>(a.g, o_tiles, (uint32_t)a.B, (uint32_t)a.heads), (uint32_t)total, per_xcd);
    return hipGetLastError();
}

template <int D, int MODE, int NW, bool PAD>
static hipError_t launch_t(const BwdArgs& a, uint32_t n_units, uint32_t n_max, hipStream_t stream) {
    constexpr uint32_t WGO = 32u * NW;
    const uint32_t o_tiles = (n_max + WGO - 1u) / WGO;
    const uint64_t total = (uint64_t)n_units * o_tiles;
    if (!fits_grid(total + 7u, 64 * NW)) return hipErrorInvalidConfiguration;
    const uint32_t per_xcd = (uint32_t)((total + 7u) / 8u);
    PadArg<PAD> pad_map;
    make_pad_arg(a.g, pad_map);
    attn_bwd_kernel<D, MODE, NW, PAD><<<8u * per_xcd, 64 * NW, 0, stream>>>(a, pad_map, make_unit_map<PAD>(a.g, o_tiles, (uint32_t)a.B, (uint32_t)a.heads), (uint32_t)total, per_xcd);
    return hipGetLastError();
}

template <int D, bool PAD>
static hipError_t launch_all(const BwdArgs& a, hipStream_t stream) {
    const uint32_t n_units = bwd_units(a);
    const UnitSizes u = unit_sizes(a.g, PAD, (uint64_t)a.B * (uint32_t)a.heads);
    const int shape = pick_bwd_shape(D, u);
    switch (shape) {
        case B128: return launch_both<D, B128, PAD>(a, n_units, u.n_max, stream);
        case B64_SPLIT: return launch_both<D, B64_SPLIT, PAD>(a, n_units, u.n_max, stream);
        case B128_SPLIT: return launch_both<D, B128_SPLIT, PAD>(a, n_units, u.n_max, stream);
        default: break;
    }
    // The dQ launch forms delta, which the second one reads.
    const hipError_t e = shape == TWO_LAUNCHES_DQ128 ? launch_t<D, BWD_DQ, 4, PAD>(a, n_units, u.n_max, stream) : launch_t<D, BWD_DQ, 8, PAD>(a, n_units, u.n_max, stream);
    return e != hipSuccess ? e : launch_t<D, BWD_DKV, 8, PAD>(a, n_units, u.n_max, stream);
}

hipError_t launch_bwd_chain_start(const BwdArgs& a, const BwdChain& w, hipStream_t stream) {
    return a.pad ? launch_delta<128, true>(a, w.n_units, w.n_steps * CHAIN_STEP, w, stream) : launch_delta<128, false>(a, w.n_units, w.n_steps * CHAIN_STEP, w, stream);
}

hipError_t launch_attn_bwd_bf16(const BwdArgs& a, hipStream_t stream) {
    if (a.head_dim == 128) return a.pad ? launch_all<128, true>(a, stream) : launch_all<128, false>(a, stream);
    if (a.head_dim == 64) return a.pad ? launch_all<64, true>(a, stream) : launch_all<64, false>(a, stream);
    return hipErrorInvalidValue;
}

}  // namespace skiparse

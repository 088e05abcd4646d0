// Host-side launchers of the HIP kernels; every function only enqueues work on `stream` and returns the
// hipError_t of the launch.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "index_map.h"
#include "wg_shape.h"

namespace skiparse {

// A dimension of a grid holds fewer than 2^32 work items.  A launch of more is not refused but cut, so the launchers refuse it.
inline bool fits_grid(uint64_t workgroups, uint32_t threads) { return workgroups * threads < 1ull << 32; }

// Sizes of the units of a launch over map g, `per_class` units (batch elements x heads) a class.
inline UnitSizes unit_sizes(const GridMap& g, bool pad, uint64_t per_class) {
    if (!pad) return {per_class * (g.mode == MODE_DENSE ? 1u : (uint32_t)(g.s * g.s)), (uint32_t)g.n_sub, (uint32_t)g.n_sub};
    const uint32_t s = (uint32_t)g.s;
    const PadMap m = make_pad_map(g);
    uint32_t rows = 0, cols = 0;  // classes that have any along either axis
    for (uint32_t p = 0; p < s; p++) {
        rows += m.hc.of(p).d != 0;
        cols += m.wc.of(p).d != 0;
    }
    return {per_class * rows * cols, make_class_map(g, m, 0, 0).n, make_class_map(g, m, s - 1u, s - 1u).n};
}

inline bool pads_most_tiles(int head_dim, const GridMap& g) {
    const uint32_t line = g.ws.d, frame = g.hpad.d / (uint32_t)g.s * line;
    return pads_most_tiles(head_dim, (uint32_t)g.n_sub, line, frame, line * (uint32_t)g.s != (uint32_t)g.W, g.hpad.d != (uint32_t)g.H_real);
}

// Row gather/scatter between the original and the sparse layout.  `to_sparse` != 0: dst is sparse.  ssp_G > 0: the sparse side is an
// all-to-all receive buffer of Sparse Sequence Parallelism with ssp_G subsequences per rank (Alg. 1, sparse_sequence_parallel, step 3).
hipError_t launch_permute(const void* src, void* dst, int B, const GridMap& g, size_t row_bytes, int to_sparse,
                          hipStream_t stream, int ssp_G = 0);

// Row moves from the sparse layout of one pattern to that of the other; g_to describes the destination pattern.
hipError_t launch_switch(const void* src, void* dst, int B, const GridMap& g_to, size_t row_bytes, hipStream_t stream);

// Flash-attention forward, bf16.  Units are (batch-like index, head); with g.mode == MODE_DENSE the batch-like
// index is a batch element of n_sub tokens, otherwise it is a subsequence (p, q, b) addressed inside the
// original layout through src_token().
struct AttnArgs {
    const void* q;
    const void* k;
    const void* v;
    void* out;
    int B;          // batch elements of the original layout
    int heads;
    int head_dim;
    float scale;    // multiplies the logits
    bool pad;       // any-resolution mode: g describes the padded grid; the kernel walks the real tokens of a class only
    GridMap g;
    // Where the output rows go.  OUT_AS_INPUT: out is addressed like q.  OUT_ORIGINAL / OUT_OTHER_PATTERN: q, k, v are the
    // sparse layout of pattern g_in (so g is a dense map over its B*s*s subsequences) and the row of query (sb, j) is written
    // at its place in the original layout / in the sparse layout of the other pattern (Alg. 1, tsa_to_gsa / gsa_to_tsa).
    float* lse;     // optional: natural-log log-sum-exp of the scaled logits of every query, [unit][position] (for the backward pass)
    int out_kind;
    int out_B;      // batch elements of the original layout (only for out_kind != OUT_AS_INPUT)
    GridMap g_in;   // index map of the input's pattern (only for out_kind != OUT_AS_INPUT)
};
enum OutKind : int { OUT_AS_INPUT = 0, OUT_ORIGINAL = 1, OUT_OTHER_PATTERN = 2 };
hipError_t launch_attn_bf16(const AttnArgs& a, hipStream_t stream);

// Flash-attention backward, bf16, in two launches: dQ and delta = rowsum(dO o O), then dK and dV; or delta, then all three gradients
// (pick_bwd_shape()).  Addressing as in AttnArgs.
enum BwdMode : int { BWD_DQ = 0, BWD_DKV = 1 };  // dQ (owner = query), dK and dV together (owner = key)
struct BwdArgs {
    const void* q;
    const void* k;
    const void* v;
    const void* out;    // the forward's output
    const void* dout;   // gradient of the loss with respect to it
    const float* lse;   // the forward's log-sum-exp, [unit][position]
    float* delta;       // workspace, [unit][position]
    void* dq;
    void* dk;
    void* dv;
    int B;
    int heads;
    int head_dim;
    float scale;
    bool pad;           // any-resolution mode, as in AttnArgs; lse and delta are laid out over the padded grid
    GridMap g;
};
inline uint32_t bwd_units(const BwdArgs& a) { return (uint32_t)a.B * (a.g.mode == MODE_DENSE ? 1u : (uint32_t)(a.g.s * a.g.s)) * (uint32_t)a.heads; }
hipError_t launch_attn_bwd_bf16(const BwdArgs& a, hipStream_t stream);

// The same gradients in one walk that passes dQ along the workgroups of a unit (attn_bwd_chain.hip): what they share in the workspace.
constexpr uint32_t CHAIN_XCCS = 16;  // values of the XCC number
// ctl: a ticket counter of every XCC, 128 bytes apart; how many groups of units are taken; every XCC's groups, 0 where not taken yet, else number + 1; every
// wavefront's progress
constexpr uint32_t CHAIN_FLAGS = 8;  // wavefronts of a workgroup
constexpr uint32_t CHAIN_NEXT = 32u * CHAIN_XCCS, CHAIN_SLOTS = CHAIN_NEXT + 32u;
constexpr uint32_t CHAIN_NONE = ~0u, CHAIN_SKIP = ~0u - 1u;  // no more work; the last group has no such unit
struct BwdChain {
    uint32_t* ctl;      // cleared by the launch that forms delta
    float* vals;        // [unit][step][2][32]: the initial logits, -lse / scale, and dP, -delta, of the queries; -inf and 0 past the end
    float* part;        // [unit][step][32 queries x head_dim] sums of dQ
    uint32_t n_units, n_blk, n_steps;              // blocks of keys and steps of the largest unit
    uint32_t together, per_group, n_groups;        // units handed out together, their blocks, and how many times
    // The work of ticket r of the group with number id (from 1): unit * n_blk + block.  Blocks come in the order of the keys, with the group's units in turn.
    __host__ __device__ uint32_t task(uint32_t id, uint32_t r) const {
        if (id > n_groups) return CHAIN_NONE;
        const uint32_t blk = r / together, unit = (id - 1u) * together + (r - blk * together);
        return unit < n_units ? unit * n_blk + blk : CHAIN_SKIP;
    }
    __host__ __device__ uint32_t n_ctl() const { return CHAIN_SLOTS + CHAIN_XCCS * (n_units + 1u) + n_units * n_blk * CHAIN_FLAGS; }
    size_t ctl_bytes() const { return ((size_t)n_ctl() * 4u + 255u) & ~(size_t)255u; }
    size_t vals_bytes() const { return (size_t)n_units * n_steps * CHAIN_STEP * 8u; }
    size_t bytes(int head_dim) const { return ctl_bytes() + vals_bytes() + (size_t)n_units * n_steps * CHAIN_STEP * (uint32_t)head_dim * 4u; }
    void place(void* at) {
        ctl = (uint32_t*)at;
        vals = (float*)((char*)at + ctl_bytes());
        part = (float*)((char*)at + ctl_bytes() + vals_bytes());
    }
};
inline BwdChain make_bwd_chain(uint32_t n_units, uint32_t n_max) {
    BwdChain w = {};
    w.n_units = n_units;
    w.n_blk = (n_max + CHAIN_OWNERS - 1u) / CHAIN_OWNERS;
    w.n_steps = (n_max + CHAIN_STEP - 1u) / CHAIN_STEP;
    w.together = chain_together(n_units, n_max);
    w.per_group = w.together * w.n_blk;
    w.n_groups = (n_units + w.together - 1u) / w.together;
    return w;
}
// Forms w.vals, clears w.ctl and marks every block of the gradients as missing, in front of the walk.
hipError_t launch_bwd_chain_start(const BwdArgs& a, const BwdChain& w, hipStream_t stream);
hipError_t launch_attn_bwd_chain(const BwdArgs& a, const BwdChain& w, hipStream_t stream);

// bf16 (original layout) -> E4M3 codes (sparse layout) + one float32 scale per (subsequence, head, 128 positions).
hipError_t launch_quantize_fp8(const void* x, void* x8, float* scales, int B, int heads, int head_dim, const GridMap& g, bool pad,
                               hipStream_t stream);

// FP8 flash-attention forward on the quantised sparse-layout tensors; bf16 output in the original layout.
struct Fp8AttnArgs {
    const void* q8;
    const void* k8;
    const void* v8;
    const float* sq;
    const float* sk;
    const float* sv;
    void* out;
    int B;            // batch elements of the original layout
    int heads;
    int head_dim;
    float scale;
    uint32_t n_blk;   // scale blocks per (subsequence, head): ceil(n_sub / 128)
    bool pad;         // any-resolution mode: g describes the padded grid; padding positions are masked keys and queries that are not stored
    GridMap g;
};
hipError_t launch_attn_fp8(const Fp8AttnArgs& a, hipStream_t stream);

}  // namespace skiparse

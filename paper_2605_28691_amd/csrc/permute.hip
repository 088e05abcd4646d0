// Row gather/scatter between the original and the sparse token order (Algorithm 1, orig_to_tsa / orig_to_gsa and
// their inverses), and between the two sparse orders.  Bound by HBM bandwidth: every row of heads*head_dim elements is contiguous in
// both layouts.  The wavefronts enumerate DESTINATION rows and find each row's source with the index map or its inverse: contiguous
// writes with gathered reads measure faster than the reverse.
//   * Longer rows: one wavefront moves one row with 16-byte accesses per lane (1 KiB contiguous per instruction).
//   * Rows up to 768 B: one wavefront moves a batch of rows.  A wavefront a row leaves most lanes idle and spends the index arithmetic, some
//     ten integer divisions, on a few hundred bytes; here lane i finds the source of row i, one evaluation for the whole batch, and
//     the batch is moved as one run of 16-byte chunks.  The rule is row_batch() in wg_shape.h.
#include "kernels.h"

namespace skiparse {

typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;

constexpr int PERMUTE_WAVES = 4;  // wavefronts per workgroup

enum RowMap : int {
    TO_SPARSE = 0,  // destination: the sparse layout, source: the original one
    TO_ORIGINAL = 1,  // the inverse
    SWITCH = 2      // destination: the sparse layout of g's pattern, source: that of the other pattern
};

// ssp_G > 0 (Sparse Sequence Parallelism, Alg. 1 sparse_sequence_parallel, step 3): the sparse side is a buffer as it arrives from the
// all-to-all, [source rank][my subsequence g'][source's subsequence g][b][position]; the algorithm's axis swap to
// [source rank][g][g'][b] = "(p q b')" order is folded into the row number instead of being a pass of its own.
__device__ inline uint32_t ssp_received_sb(uint32_t sb, uint32_t B, uint32_t G) {
    const uint32_t b = B / G;                        // batch elements per subsequence
    const uint32_t pq = sb / B, bi = sb - pq * B;    // class of the source pattern; (g', batch element)
    const uint32_t r = pq / G, gs = pq - r * G, gd = bi / b, bb = bi - gd * b;
    return ((r * G + gd) * G + gs) * b + bb;
}

// token (b, t*H + h, w) -> its row in the sparse layout of one pattern (Alg. 1 read backwards; H and W are multiples of s for the
// token-wise pattern and of s*s for the group-wise one, so t*H + h splits like h)
__device__ inline uint32_t sparse_row_of(bool group, uint32_t s, uint32_t W, uint32_t n_sub, uint32_t B, uint32_t b, uint32_t n, uint32_t ssp_G) {
    const uint32_t th = n / W, w = n - th * W;
    uint32_t p, q, r, ws;
    if (group) {
        p = (th / s) % s;
        q = (w / s) % s;
        r = (th / (s * s)) * s + th % s;
        ws = (w / (s * s)) * s + w % s;
    } else {
        p = th % s;
        q = w % s;
        r = th / s;
        ws = w / s;
    }
    uint32_t sb = (p * s + q) * B + b;
    if (ssp_G) sb = ssp_received_sb(sb, B, ssp_G);
    return sb * n_sub + r * (W / s) + ws;
}

// row number in the source of destination row `row`
template <int MAP>
__device__ inline uint32_t source_row(const GridMap& g, uint32_t B, uint32_t row, uint32_t ssp_G) {
    const uint32_t s = (uint32_t)g.s, W = (uint32_t)g.W, n_sub = (uint32_t)g.n_sub;
    if (MAP == TO_ORIGINAL) {
        if (g.mode == MODE_DENSE) return row;
        const uint32_t b = row / (uint32_t)g.n_tok;
        return sparse_row_of(g.mode == MODE_GROUP, s, W, n_sub, B, b, row - b * (uint32_t)g.n_tok, ssp_G);
    }
    const uint32_t sb = row / n_sub, j = row - sb * n_sub;
    const uint32_t pq = sb / B, b = sb - pq * B;
    const uint32_t p = pq / s, tok = src_token(g, p, pq - p * s, j);
    return MAP == SWITCH ? sparse_row_of(g.mode != MODE_GROUP, s, W, n_sub, B, b, tok, 0u) : b * (uint32_t)g.n_tok + tok;
}

template <int MAP, int UNROLL>
__global__ __launch_bounds__(PERMUTE_WAVES * 64) void permute_rows_kernel(const u32x4* __restrict__ src, u32x4* __restrict__ dst, int B, GridMap g,
                                                                       uint32_t chunks_per_row, uint32_t n_rows, uint32_t ssp_G) {
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t row = blockIdx.x * PERMUTE_WAVES + (threadIdx.x >> 6);
    if (row >= n_rows) return;
    const u32x4* s = src + (size_t)source_row<MAP>(g, (uint32_t)B, row, ssp_G) * chunks_per_row;
    u32x4* d = dst + (size_t)row * chunks_per_row;
    uint32_t c = lane;
    for (; c + (UNROLL - 1) * 64u < chunks_per_row; c += UNROLL * 64u) {
        u32x4 tmp[UNROLL];
#pragma unroll
        for (int u = 0; u < UNROLL; u++) tmp[u] = __builtin_nontemporal_load(s + c + u * 64u);
#pragma unroll
        for (int u = 0; u < UNROLL; u++) __builtin_nontemporal_store(tmp[u], d + c + u * 64u);
    }
    for (; c < chunks_per_row; c += 64u) __builtin_nontemporal_store(__builtin_nontemporal_load(s + c), d + c);
}

constexpr int BATCH_UNROLL = BATCH_CHUNKS / 64;  // a full batch in one round of loads
static_assert(BATCH_UNROLL * 64 == BATCH_CHUNKS, "whole rounds of the wavefront");

template <int MAP>
__global__ __launch_bounds__(PERMUTE_WAVES * 64) void permute_short_rows_kernel(const u32x4* __restrict__ src, u32x4* __restrict__ dst, int B, GridMap g,
                                                                             FastDiv chunks, uint32_t n_rows, uint32_t batch, uint32_t ssp_G) {
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t row0 = (blockIdx.x * PERMUTE_WAVES + (threadIdx.x >> 6)) * batch;  // n_rows < 2^31: no overflow
    if (row0 >= n_rows) return;
    const uint32_t n = n_rows - row0 < batch ? n_rows - row0 : batch;  // at most 64
    const uint32_t from = source_row<MAP>(g, (uint32_t)B, row0 + (lane < n ? lane : n - 1u), ssp_G);
    u32x4* const d = dst + (size_t)row0 * chunks.d;
    const uint32_t total = n * chunks.d;  // at most BATCH_CHUNKS: the division below is exact
    u32x4 tmp[BATCH_UNROLL];
#pragma unroll
    for (int k = 0; k < BATCH_UNROLL; k++) {
        const uint32_t u = k * 64u + lane, uc = u < total ? u : total - 1u;  // lanes past the end repeat the last chunk and store nothing
        const uint32_t i = chunks.div(uc), c = uc - i * chunks.d;
        tmp[k] = __builtin_nontemporal_load(src + (size_t)(uint32_t)__shfl((int)from, (int)i) * chunks.d + c);
    }
#pragma unroll
    for (int k = 0; k < BATCH_UNROLL; k++) {
        const uint32_t u = k * 64u + lane;
        if (u < total) __builtin_nontemporal_store(tmp[k], d + u);
    }
}

template <int MAP, int UNROLL>
static void launch_long(const void* src, void* dst, int B, const GridMap& g, uint32_t chunks, uint32_t n_rows, uint32_t ssp_G, hipStream_t stream) {
    const uint32_t blocks = (n_rows + PERMUTE_WAVES - 1) / PERMUTE_WAVES;
    permute_rows_kernel<MAP, UNROLL><<<blocks, PERMUTE_WAVES * 64, 0, stream>>>((const u32x4*)src, (u32x4*)dst, B, g, chunks, n_rows, ssp_G);
}

template <int MAP>
static hipError_t launch_rows(const void* src, void* dst, int B, const GridMap& g, size_t row_bytes, uint32_t ssp_G, hipStream_t stream) {
    const uint32_t chunks = (uint32_t)(row_bytes / 16);
    const uint32_t s2 = g.mode == MODE_DENSE ? 1u : (uint32_t)(g.s * g.s);
    const uint32_t n_rows = (uint32_t)B * s2 * (uint32_t)g.n_sub;
    const uint32_t batch = row_batch(chunks, n_rows);
    if (batch > 1u) {
        const uint32_t per_block = batch * PERMUTE_WAVES, blocks = (n_rows + per_block - 1) / per_block;
        permute_short_rows_kernel<MAP><<<blocks, PERMUTE_WAVES * 64, 0, stream>>>((const u32x4*)src, (u32x4*)dst, B, g, make_fastdiv32(chunks), n_rows, batch, ssp_G);
    } else if (chunks >= 5 * 64) {
        launch_long<MAP, 5>(src, dst, B, g, chunks, n_rows, ssp_G, stream);
    } else if (chunks >= 3 * 64) {
        launch_long<MAP, 3>(src, dst, B, g, chunks, n_rows, ssp_G, stream);
    } else {
        launch_long<MAP, 1>(src, dst, B, g, chunks, n_rows, ssp_G, stream);
    }
    return hipGetLastError();
}

hipError_t launch_switch(const void* src, void* dst, int B, const GridMap& g_to, size_t row_bytes, hipStream_t stream) {
    return launch_rows<SWITCH>(src, dst, B, g_to, row_bytes, 0u, stream);
}

hipError_t launch_permute(const void* src, void* dst, int B, const GridMap& g, size_t row_bytes, int to_sparse,
                          hipStream_t stream, int ssp_G) {
    return to_sparse ? launch_rows<TO_SPARSE>(src, dst, B, g, row_bytes, 0u, stream) : launch_rows<TO_ORIGINAL>(src, dst, B, g, row_bytes, (uint32_t)ssp_G, stream);
}

}  // namespace skiparse

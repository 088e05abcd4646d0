// Row gather/scatter between the original and the sparse token order (Algorithm 1, orig_to_tsa / orig_to_gsa and
// their inverses), and between the two sparse orders.  Bound by HBM bandwidth: every row of heads*head_dim elements is contiguous in
// both layouts.  The wavefronts enumerate DESTINATION rows and find each row's source with the index map or its inverse: contiguous
// writes with gathered reads measure faster than the reverse.
//   * Longer rows: one wavefront moves 1 KiB of a row, one 16-byte access a lane, and the next ones the rest of it.  What is in flight then
//     lies close together (8 MB on the whole chip, not 80), and the copy runs at 6.5 TB/s; a wavefront a row of 10 KiB with five loads in
//     flight reached 5.7, with two 6.2.  Every wavefront forms its row number anew, so the divisions are multiplications on the scalar unit
//     (Div32): with the compiler's own they bound the copy (permute, switch and unpermute of 80,640 rows of 10 KiB 872 us, in parts of 1 KiB
//     795, with Div32 756).  Rows that fill the last 1 KiB badly go in parts of up to 2 KiB: row_unroll() in wg_shape.h.
//   * Rows up to 768 B: one wavefront moves a batch of rows.  A wavefront a row leaves most lanes idle and spends the index arithmetic, some
//     ten integer divisions, on a few hundred bytes; here lane i finds the source of row i, one evaluation for the whole batch, and
//     the batch is moved as one run of 16-byte chunks.  The rule is row_batch() in wg_shape.h.
#include "kernels.h"

namespace skiparse {

typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;

constexpr int PERMUTE_WAVES = 4;  // wavefronts per workgroup

template <int MAP, int UNROLL>
__global__ __launch_bounds__(PERMUTE_WAVES * 64) void permute_rows_kernel(const u32x4* __restrict__ src, u32x4* __restrict__ dst, RowArgs g, Div32 parts,
                                                                          uint32_t span, uint32_t chunks, uint32_t n_rows, uint32_t ssp_G) {
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t id = __builtin_amdgcn_readfirstlane(blockIdx.x * PERMUTE_WAVES + (threadIdx.x >> 6));
    const uint32_t row = parts.div(id), part = id - row * parts.d;
    if (row >= n_rows) return;
    const u32x4* s = src + (size_t)source_row<MAP>(g, row, ssp_G) * chunks;
    u32x4* d = dst + (size_t)row * chunks;
    const uint32_t from = part * span, to = from + span < chunks ? from + span : chunks;
    for (uint32_t c = from + lane; c < to; c += UNROLL * 64u) {  // one round, but for tensors of more than MAX_ROW_WAVES spans
        u32x4 tmp[UNROLL];
#pragma unroll
        for (int u = 0; u < UNROLL; u++)
            if (u == 0 || c + u * 64u < to) tmp[u] = __builtin_nontemporal_load(s + c + u * 64u);
#pragma unroll
        for (int u = 0; u < UNROLL; u++)
            if (u == 0 || c + u * 64u < to) __builtin_nontemporal_store(tmp[u], d + c + u * 64u);
    }
}

static_assert(BATCH_CHUNKS == 4 * 64, "a full batch in one round of four loads a lane");

// UNROLL: loads a lane that the launch's batches need
template <int MAP, int UNROLL>
__global__ __launch_bounds__(PERMUTE_WAVES * 64) void permute_short_rows_kernel(const u32x4* __restrict__ src, u32x4* __restrict__ dst, RowArgs g,
                                                                             FastDiv chunks, uint32_t n_rows, uint32_t batch, uint32_t ssp_G) {
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t row0 = (blockIdx.x * PERMUTE_WAVES + (threadIdx.x >> 6)) * batch;  // n_rows < 2^31: no overflow
    if (row0 >= n_rows) return;
    const uint32_t n = n_rows - row0 < batch ? n_rows - row0 : batch;  // at most 64
    const uint32_t from = source_row<MAP>(g, row0 + (lane < n ? lane : n - 1u), ssp_G);
    u32x4* const d = dst + (size_t)row0 * chunks.d;
    const uint32_t total = n * chunks.d;  // at most 64 * UNROLL: the division below is exact
    u32x4 tmp[UNROLL];
#pragma unroll
    for (int k = 0; k < UNROLL; k++) {
        const uint32_t u = k * 64u + lane, uc = u < total ? u : total - 1u;  // lanes past the end repeat the last chunk and store nothing
        const uint32_t i = chunks.div(uc), c = uc - i * chunks.d;
        tmp[k] = __builtin_nontemporal_load(src + (size_t)(uint32_t)__shfl((int)from, (int)i) * chunks.d + c);
    }
#pragma unroll
    for (int k = 0; k < UNROLL; k++) {
        const uint32_t u = k * 64u + lane;
        if (u < total) __builtin_nontemporal_store(tmp[k], d + u);
    }
}

template <int MAP, int UNROLL>
static hipError_t launch_long(const void* src, void* dst, const RowArgs& g, uint32_t chunks, uint32_t n_rows, uint32_t ssp_G, hipStream_t stream) {
    const uint32_t span = row_span(chunks, n_rows, UNROLL), parts = (chunks + span - 1u) / span;
    const uint64_t blocks = ((uint64_t)n_rows * parts + PERMUTE_WAVES - 1) / PERMUTE_WAVES;
    if (!fits_grid(blocks, PERMUTE_WAVES * 64)) return hipErrorInvalidConfiguration;
    permute_rows_kernel<MAP, UNROLL><<<(uint32_t)blocks, PERMUTE_WAVES * 64, 0, stream>>>((const u32x4*)src, (u32x4*)dst, g, make_div32(parts), span, chunks, n_rows, ssp_G);
    return hipGetLastError();
}

template <int MAP, int UNROLL>
static hipError_t launch_short(const void* src, void* dst, const RowArgs& g, uint32_t chunks, uint32_t n_rows, uint32_t batch, uint32_t ssp_G, hipStream_t stream) {
    const uint32_t per_block = batch * PERMUTE_WAVES, blocks = (n_rows + per_block - 1) / per_block;
    if (!fits_grid(blocks, PERMUTE_WAVES * 64)) return hipErrorInvalidConfiguration;
    permute_short_rows_kernel<MAP, UNROLL><<<blocks, PERMUTE_WAVES * 64, 0, stream>>>((const u32x4*)src, (u32x4*)dst, g, make_fastdiv32(chunks), n_rows, batch, ssp_G);
    return hipGetLastError();
}

template <int MAP>
static hipError_t launch_rows(const void* src, void* dst, int B, const GridMap& g, size_t row_bytes, uint32_t ssp_G, hipStream_t stream) {
    const uint32_t chunks = (uint32_t)(row_bytes / 16);
    const uint32_t s2 = g.mode == MODE_DENSE ? 1u : (uint32_t)(g.s * g.s);
    const uint32_t n_rows = (uint32_t)B * s2 * (uint32_t)g.n_sub;
    const uint32_t batch = row_batch(chunks, n_rows);
    const RowArgs args = make_row_args<MAP>(g, (uint32_t)B);
    if (batch > 1u) {
        // few rows or very short ones: no more rounds than the batch has (three moves of 4608 rows of 16 to 512 B 8.3..9.9 us -> 7.7..9.2)
        const uint32_t per_wave = batch * chunks;
        if (per_wave <= 64u) return launch_short<MAP, 1>(src, dst, args, chunks, n_rows, batch, ssp_G, stream);
        if (per_wave <= 128u) return launch_short<MAP, 2>(src, dst, args, chunks, n_rows, batch, ssp_G, stream);
        return launch_short<MAP, 4>(src, dst, args, chunks, n_rows, batch, ssp_G, stream);
    }
    return row_unroll(chunks) == 2u ? launch_long<MAP, 2>(src, dst, args, chunks, n_rows, ssp_G, stream) : launch_long<MAP, 1>(src, dst, args, chunks, n_rows, ssp_G, stream);
}

hipError_t launch_switch(const void* src, void* dst, int B, const GridMap& g_to, size_t row_bytes, hipStream_t stream) {
    return launch_rows<SWITCH>(src, dst, B, g_to, row_bytes, 0u, stream);
}

hipError_t launch_permute(const void* src, void* dst, int B, const GridMap& g, size_t row_bytes, int to_sparse,
                          hipStream_t stream, int ssp_G) {
    return to_sparse ? launch_rows<TO_SPARSE>(src, dst, B, g, row_bytes, 0u, stream) : launch_rows<TO_ORIGINAL>(src, dst, B, g, row_bytes, (uint32_t)ssp_G, stream);
}

}  // namespace skiparse

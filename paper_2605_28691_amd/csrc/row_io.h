// How the attention kernels move the rows that a wavefront owns.
//
// Results leave through LDS.  In the accumulator layout a lane holds 4 consecutive channels of its row here and 4 there: stored
// from there, an instruction of a wavefront writes 16 bytes to each of 32 rows, and the address unit takes such pieces one after the other.  So a wavefront
// lays the channels down in LDS (a region of its own, no barrier) and stores whole 128-byte lines (64 where it has 32 channels), 8 rows an instruction.
// Clocks of a workgroup from its last product until its stores have arrived, before -> after: 4 wavefronts at head_dim 128 (48 units of 390 tokens) 4990 ->
// 2640, 8 (48 of 8190) 7510 -> 3400, dK and dV of 128 keys (48 of 400) 4950 -> 3070; two wavefronts a compute unit, where nothing queues, 1310 -> 1790 (units
// that short store their rows directly, see FWD_DIRECT_ROWS and BWD_DIRECT_ROWS).
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "lds_layout.h"

namespace skiparse {

// Where the 32 rows of a wavefront go, CH channels at a time: a pass over them takes N instructions, instruction i rows RPI*i ...
template <int CH>
struct RowDest {
    static_assert(CH == 64 || CH == 32, "channels of a pass");
    static constexpr int LPR = CH / 8, RPI = 64 / LPR, N = 32 / RPI;  // lanes a row, rows an instruction, instructions
    size_t off[N];  // elements
    bool ok[N];
    // row: number of the row that lane l % 32 owns (below 2^32: a row has 128 bytes at least), row_len: elements a row; bit r of `stored`: row r is stored
    __device__ __attribute__((always_inline)) inline RowDest(uint32_t row, size_t row_len, uint32_t stored, uint32_t lane) {
#pragma unroll
        for (int i = 0; i < N; i++) {
            const uint32_t r = RPI * i + lane / LPR;
            off[i] = (size_t)(uint32_t)__shfl((int)row, (int)r) * row_len;
            ok[i] = (stored >> r & 1u) != 0;
        }
    }
};

// acc * f, rounded to bf16, to dst + row offset: register 4*g + e of block mt is channel 32*mt + 8*g + 4*(lane/32) + e of row lane % 32.
// buf: ROWS * CH * 2 bytes of LDS of the wavefront's own, 16-byte aligned.  Chunk c (8 channels) of row r lies at another position of the row, and with 64
// channels its halves are exchanged in every other run of 8 rows, so that no two of 16 lanes
// write to one bank, 8 bytes each, and 16 lanes' 16-byte reads touch every bank once.
template <int CH, int ROWS, int BLOCKS>
__device__ __attribute__((always_inline)) inline void store_rows(char* buf, const __attribute__((ext_vector_type(16))) float (&acc)[BLOCKS], float f, __bf16* dst, const RowDest<CH>& d, uint32_t lane) {
    static_assert(ROWS % RowDest<CH>::RPI == 0 && 32 % ROWS == 0 && BLOCKS * 32 % CH == 0, "whole passes");
    typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
    typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
    constexpr int LPR = RowDest<CH>::LPR, RPI = RowDest<CH>::RPI;
    const uint32_t r = lane & 31u, h = lane >> 5;
    auto swz = [](uint32_t row) __attribute__((always_inline)) -> uint32_t { return CH == 64 ? row & 7u : row >> 2 & 3u; };
    char* const wr = buf + (r & (uint32_t)(ROWS - 1)) * (2u * CH) + 8u * (CH == 64 ? h ^ (r >> 3 & 1u) : h);
    const char* const rd = buf + lane / LPR * (2u * CH) + ((lane % LPR) ^ swz(lane / LPR)) * 16u;
    __bf16* const out = dst + lane % LPR * 8u;
    // other lanes may have read the region last; the wavefront's LDS accesses take effect in order, and the fences keep the compiler from exchanging them
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int part = 0; part < 32 / ROWS; part++)
#pragma unroll
        for (int c = 0; c < BLOCKS * 32 / CH; c++) {
            if (ROWS == 32 || r / ROWS == (uint32_t)part) {
#pragma unroll
                for (int k = 0; k < LPR; k++) {
                    bf16x4 o;
#pragma unroll
                    for (int e = 0; e < 4; e++) o[e] = (__bf16)(acc[c * CH / 32 + k / 4][4 * (k % 4) + e] * f);
                    *(bf16x4*)(wr + (((uint32_t)k ^ swz(r)) * 16u)) = o;
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int i = 0; i < ROWS / RPI; i++) {
                const u32x4 x = *(const u32x4*)(rd + i * 1024);
                const int n = part * (ROWS / RPI) + i;
                const u32x4 y = CH == 32 || n % 2 == 0 ? x : u32x4{x[2], x[3], x[0], x[1]};
                if (d.ok[n]) *(u32x4*)(out + d.off[n] + c * CH) = y;
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
        }
}

// The same from where the channels are: row, row_len as in RowDest, `row` being the lane's own.  For workgroups of few rows, whose stores do not queue and which
// the way through LDS only delays.
template <int BLOCKS>
__device__ __attribute__((always_inline)) inline void store_own_row(const __attribute__((ext_vector_type(16))) float (&acc)[BLOCKS], float f, __bf16* dst, uint32_t row, size_t row_len, uint32_t lane) {
    typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
    asm volatile("" : "+v"(row), "+v"(lane));  // formed here: else the address is kept in registers through the whole walk (3 spilled values in the backward's B128)
    __bf16* const at = dst + (size_t)row * row_len + (lane >> 5) * 4u;
#pragma unroll
    for (int mt = 0; mt < BLOCKS; mt++)
#pragma unroll
        for (int g = 0; g < 4; g++) {
            bf16x4 o;
#pragma unroll
            for (int e = 0; e < 4; e++) o[e] = (__bf16)(acc[mt][4 * g + e] * f);
            *(bf16x4*)(at + mt * 32 + g * 8) = o;
        }
}

// Rows of a workgroup up to which they are moved directly, and, in the forward, queries loaded as fragments.  us in a row, through LDS / directly, head_dim 128:
// forward, 4 units of 16 tokens 4.47 / 3.93, of 32 4.41 / 4.04, of 40 5.12 / 4.82 (200 of 56: 5.32 / 5.45); backward, 4 of 16 7.26 / 6.94, of 32 7.47 / 7.20, but 200 of
// 40 11.6 / 12.4; 8-bit, 8 of 32 5.2 / 4.8.
constexpr uint32_t FWD_DIRECT_ROWS = 48, BWD_DIRECT_ROWS = 32;

// The way in: a wavefront's 32 rows as B operands (lane = row lane % 32, 8 consecutive channels starting at 16*ks + 8*(lane/32)).  Loaded in that shape an
// instruction takes 32 bytes of each of 32 rows; here it takes 128 bytes of 8, and the fragments are picked up from LDS.  Forward calls, us, loaded as fragments ->
// so: 12 units of 132 tokens 8.06 -> 7.94, 9.32 -> 9.01 and 13.16 -> 12.91 in chains, 48 of 390 12.39 -> 12.34.  The backward kernels load fragments: with this
// their registers are allotted another way, and the whole training step of 48 units of 8190 tokens takes 6560 instead of 6200.
template <int D>
struct RowLoad {
    typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
    static constexpr int NC = D / 64;
    bf16x8 x[NC][4];
    // row, row_len as in RowDest; src: the unit's first row
    __device__ __attribute__((always_inline)) inline void issue(const __bf16* src, uint32_t row, size_t row_len, uint32_t lane) {
#pragma unroll
        for (int i = 0; i < 4; i++) {
            const __bf16* const at = src + (size_t)(uint32_t)__shfl((int)row, (int)(8 * i + (lane >> 3))) * row_len + (lane & 7u) * 8u;
#pragma unroll
            for (int c = 0; c < NC; c++) x[c][i] = *(const bf16x8*)(at + c * 64);
        }
    }
    // buf: ROWS * 128 bytes of LDS of the wavefront's own.  Rows of 64 channels in the layout of a head_dim 64 tile.
    template <int ROWS>
    __device__ __attribute__((always_inline)) inline void fragments(char* buf, bf16x8 (&f)[D / 16], uint32_t lane) const {
        static_assert(ROWS == 32 || ROWS == 16, "rows of a pass");
        const uint32_t r = lane & 31u, h = lane >> 5;
        char* const wr = buf + (lane >> 3) * 128u;  // rows 8 apart differ in the swizzle
        const char* const rd = buf + (r & (uint32_t)(ROWS - 1)) * 128u;
#pragma unroll
        for (int c = 0; c < NC; c++)
#pragma unroll
            for (int part = 0; part < 32 / ROWS; part++) {
#pragma unroll
                for (int i = 0; i < ROWS / 8; i++)
                    *(bf16x8*)(wr + i * 1024 + (((lane & 7u) ^ lds_swizzle<64>(8u * i + (lane >> 3))) * 16u)) = x[c][part * (ROWS / 8) + i];
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                __builtin_amdgcn_wave_barrier();
                if (ROWS == 32 || r / ROWS == (uint32_t)part) {
#pragma unroll
                    for (int k = 0; k < 4; k++) f[4 * c + k] = *(const bf16x8*)(rd + (((2u * k + h) ^ lds_swizzle<64>(r)) * 16u));
                }
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                __builtin_amdgcn_wave_barrier();
            }
    }
};

// of the 32 rows from `first`, those below n
__host__ __device__ inline uint32_t rows_below(uint32_t first, uint32_t n) {
    return first >= n ? 0u : n - first >= 32u ? ~0u : (1u << (n - first)) - 1u;
}

}  // namespace skiparse

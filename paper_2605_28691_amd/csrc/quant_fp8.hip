// bf16 -> FP8 E4M3 block quantisation fused with the Skiparse rearrangement (8-bit variant of the attention path).
//
// One workgroup handles one (subsequence, head, block of 128 consecutive positions): it gathers the block's rows from
// the original layout (Algorithm 1 index map), takes max |x| over the block, and writes
//     code = e4m3( clamp( x * (448 / amax), -448, 448 ) )     scale = amax / 448      (1 and 1 if amax = 0)
// in the sparse layout.  All decisions are taken in float32.  Bound by HBM bandwidth: 2 bytes read and 1 byte written
// per element, every row segment (head_dim bf16 values) read as whole 16-byte chunks.  Small tensors are bound by the index arithmetic before the first
// load: one evaluation of the map a wavefront, lane = row, and the workgroup's own numbers on the scalar unit (Div32); three tensors of 8 MB with
// an evaluation a row and pass 23.6 us, so 19.1, in an order that the caches can use 16.5; of 826 MB 692 -> 628 (5.9 TB/s).
#include "kernels.h"

namespace skiparse {

typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;
typedef __attribute__((ext_vector_type(2))) unsigned int u32x2;

constexpr int QBLOCK = 128;  // positions per scale block

struct QuantArgs {
    Div32 n_blk, heads, B, s;  // divisions that take a workgroup's number apart, on the scalar unit
};

// PAD: any-resolution mode (Sec. 3.2): positions run over the grid padded to multiples of s*s; a padding position is a row of zero
// codes and does not enter the block's maximum.
template <int D, bool PAD, bool READ_ONCE, bool STREAM_OUT>
__global__ __launch_bounds__(256) void quantize_fp8_kernel(const unsigned short* __restrict__ x, unsigned char* __restrict__ x8,
                                                           float* __restrict__ scales, QuantArgs a, GridMap g) {
    constexpr int CH = D / 8;        // 16-byte chunks per row segment
    constexpr int RPI = 64 / CH;     // rows a wavefront covers at once
    constexpr int PASSES = 32 / RPI; // a wavefront takes 32 rows of the block, RPI of every 4 * RPI: short units have some
                                     // for each (224 units of 32 positions at head_dim 128, 32 rows in a run 3.63 us, so 3.11)
    __shared__ float wave_max[4];
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // every XCD takes a contiguous range, heads fastest: what is in flight on it lies close together, and the segments of neighbouring heads meet
    // in its L2 (a head's segment of codes is half a line at head_dim 64)
    const uint32_t per_xcd = gridDim.x / 8u;
    const uint32_t id = blockIdx.x < per_xcd * 8u ? (blockIdx.x & 7u) * per_xcd + (blockIdx.x >> 3) : blockIdx.x;
    const uint32_t t = a.heads.div(id), head = id - t * a.heads.d;
    const uint32_t sb = a.n_blk.div(t), blk = t - sb * a.n_blk.d, uh = sb * a.heads.d + head;
    const uint32_t pq = a.B.div(sb), b = sb - pq * a.B.d, p = a.s.div(pq), q = pq - p * a.s.d;  // (dense: s = 1, one class)
    const uint32_t n_sub = (uint32_t)g.n_sub, C = a.heads.d * D;  // elements per token
    const uint32_t j0 = blk * QBLOCK + wave * RPI;  // position of row i of the wavefront: j0 + i / RPI * (4 * RPI) + i % RPI

    // lane i finds the token of row i of the wavefront's 32; NONE: past the end, or padding
    constexpr uint32_t NONE = 0xffffffffu;
    uint32_t tok = NONE;
    {
        const uint32_t j = j0 + (lane & 31u) / RPI * (4u * RPI) + lane % RPI;
        bool real = true;
        const uint32_t n = PAD ? src_token_padded(g, p, q, j < n_sub ? j : 0u, &real) : src_token(g, p, q, j < n_sub ? j : 0u);
        if (j < n_sub && real) tok = n;
    }
    const uint32_t c = lane % CH, r0 = lane / CH;
    const unsigned short* xb = x + (size_t)b * (uint32_t)g.n_tok * C + head * D + c * 8u;
    u32x4 v[PASSES];
#pragma unroll
    for (int ps = 0; ps < PASSES; ps++) {
        const uint32_t n = (uint32_t)__shfl((int)tok, (int)(ps * RPI + r0));
        const u32x4* src = (const u32x4*)(xb + (uint64_t)n * C);
        v[ps] = u32x4{0u, 0u, 0u, 0u};
        if (n != NONE) v[ps] = READ_ONCE ? __builtin_nontemporal_load(src) : *src;
    }
    float amax = 0.f;
#pragma unroll
    for (int ps = 0; ps < PASSES; ps++)
#pragma unroll
        for (int e = 0; e < 4; e++) {
            amax = fmaxf(amax, fabsf(__uint_as_float(v[ps][e] << 16)));          // low bf16 of the dword
            amax = fmaxf(amax, fabsf(__uint_as_float(v[ps][e] & 0xffff0000u)));  // high bf16
        }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) amax = fmaxf(amax, __shfl_xor(amax, off));
    if (lane == 0) wave_max[wave] = amax;
    __syncthreads();
    amax = fmaxf(fmaxf(wave_max[0], wave_max[1]), fmaxf(wave_max[2], wave_max[3]));
    const float inv = amax > 0.f ? 448.0f / amax : 1.0f;
    if (tid == 0) scales[(size_t)uh * a.n_blk.d + blk] = amax > 0.f ? amax / 448.0f : 1.0f;

    unsigned char* dst = x8 + ((size_t)sb * n_sub + j0 + r0) * C + head * D + c * 8u;
#pragma unroll
    for (int ps = 0; ps < PASSES; ps++, dst += (size_t)(4 * RPI) * C) {
        if (j0 + ps * (4 * RPI) + r0 >= n_sub) continue;
        u32x2 out;
#pragma unroll
        for (int e = 0; e < 4; e += 2) {  // dwords e, e+1 hold elements 2e..2e+3 -> four codes = one output dword
            const float x0 = fminf(fmaxf(__uint_as_float(v[ps][e] << 16) * inv, -448.0f), 448.0f);
            const float x1 = fminf(fmaxf(__uint_as_float(v[ps][e] & 0xffff0000u) * inv, -448.0f), 448.0f);
            const float x2 = fminf(fmaxf(__uint_as_float(v[ps][e + 1] << 16) * inv, -448.0f), 448.0f);
            const float x3 = fminf(fmaxf(__uint_as_float(v[ps][e + 1] & 0xffff0000u) * inv, -448.0f), 448.0f);
            int pk = __builtin_amdgcn_cvt_pk_fp8_f32(x0, x1, 0, false);  // codes of x0, x1 into the low half
            pk = __builtin_amdgcn_cvt_pk_fp8_f32(x2, x3, pk, true);      // codes of x2, x3 into the high half
            out[e >> 1] = (uint32_t)pk;
        }
        if (STREAM_OUT) __builtin_nontemporal_store(out, (u32x2*)dst);
        else *(u32x2*)dst = out;
    }
}

template <int D, bool PAD>
static hipError_t launch_quantize_t(const void* x, void* x8, float* scales, const QuantArgs& a, const GridMap& g, uint32_t blocks, uint64_t bytes, hipStream_t stream) {
    const unsigned short* xs = (const unsigned short*)x;
    unsigned char* x8c = (unsigned char*)x8;
    // Which side goes past the caches (three tensors, us; loads cached + stores past / loads past + stores cached / both past).  What a program has
    // just written is still in the 256 MB cache if it is small: 8 MB 16.5 / 18.4 / 19.7, 32 MB 31.9 / 37.7 / 38.2; larger inputs only displace the codes
    // that attention reads next: 100 MB 90.7 / 82.2 / 87.1, 200 MB 175 / 157 / 169, 248 MB at head_dim 64 226 / 189 / 226; codes of more than that
    // are not there either: 826 MB 652 / 660 / 628.
    if (bytes <= (64ull << 20)) quantize_fp8_kernel<D, PAD, false, true><<<blocks, 256, 0, stream>>>(xs, x8c, scales, a, g);
    else if (bytes <= (512ull << 20)) quantize_fp8_kernel<D, PAD, true, false><<<blocks, 256, 0, stream>>>(xs, x8c, scales, a, g);
    else quantize_fp8_kernel<D, PAD, true, true><<<blocks, 256, 0, stream>>>(xs, x8c, scales, a, g);
    return hipGetLastError();
}

hipError_t launch_quantize_fp8(const void* x, void* x8, float* scales, int B, int heads, int head_dim, const GridMap& g, bool pad,
                               hipStream_t stream) {
    const uint32_t s = g.mode == MODE_DENSE ? 1u : (uint32_t)g.s;
    const uint32_t n_blk = ((uint32_t)g.n_sub + QBLOCK - 1) / QBLOCK;
    const uint64_t blocks = (uint64_t)B * s * s * (uint32_t)heads * n_blk;
    if (!fits_grid(blocks, 256u)) return hipErrorInvalidConfiguration;
    const QuantArgs a = {make_div32(n_blk), make_div32((uint32_t)heads), make_div32((uint32_t)B), make_div32(s)};
    const uint64_t bytes = (uint64_t)B * (uint32_t)g.n_tok * (uint32_t)heads * (uint32_t)head_dim * 2u;
    if (head_dim == 128)
        return pad ? launch_quantize_t<128, true>(x, x8, scales, a, g, (uint32_t)blocks, bytes, stream)
                   : launch_quantize_t<128, false>(x, x8, scales, a, g, (uint32_t)blocks, bytes, stream);
    if (head_dim == 64)
        return pad ? launch_quantize_t<64, true>(x, x8, scales, a, g, (uint32_t)blocks, bytes, stream)
                   : launch_quantize_t<64, false>(x, x8, scales, a, g, (uint32_t)blocks, bytes, stream);
    return hipErrorInvalidValue;
}

}  // namespace skiparse

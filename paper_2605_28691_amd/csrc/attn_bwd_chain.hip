// bf16 flash-attention backward for gfx950, all three gradients in ONE walk: the five matrix products of the definition,
//     S = Q K^T,  dP = dO V^T,  dV += P^T dO,  dK += dS^T Q,  dQ += dS K
// where attn_bwd.hip, whose dQ and dK+dV owners each form S and dP for themselves, takes seven.  A workgroup owns 256 keys (a lane one of them, as in the dK+dV
// part there) and walks all queries of the unit, 32 a step.  dK and dV are accumulated in registers.  dQ of a step is a sum over ALL keys, so it is passed along
// the unit's workgroups: workgroup i takes the float32 sums that workgroup i-1 has left for these 32 queries, starts its accumulators with them, adds the
// products over its own 256 keys, and leaves them for workgroup i+1; the last one rounds them to bf16 into dq.  No atomics on the sums and one order, that of
// the keys: the result is deterministic.
//   * Why: at 160 units of 20,160 tokens the two launches take 41 ms (dQ) and 54 (dK+dV) of matrix products at the board's power limit, two sevenths of them S and dP
//     formed a second time; one walk takes 80 (1040 TFLOP/s on the definition), 48 units of 8190 tokens 4.1 instead of 4.65.
//   * What bounds it: a step takes about 4850 clocks at 1.88 GHz, 2560 of which are the 80 products of a SIMD (matrix pipe 53 % busy, LDS 48, vector ALU 32).  The clock
//     is down, but the power limit is not all: busy x clock is 0.99 GHz where the two launches reach 1.17 and 1.19, and on zeros, at 2.38 GHz, a step takes 5300 clocks (69.5
//     ms; the two launches 70.5): it waits for memory, which the clock does not speed up.  Without the sums' way through memory it took 74.7 ms where it took 85.
//   * A unit's workgroups run on ONE XCD, whose L2 the sums pass through: workgroups take their work from a queue of the XCD that they find themselves on, so
//     that no placement is assumed.  A store is there for the XCD's other CUs once vmcnt says so (the vector L1 writes through); the reader's loads go past its own
//     L1.  Of 130 GB of sums about a fifth leave the L2 (28.6 GB written).
//   * The sums are asked for between the products of dV of the step before (the flag that allows them at that step's start) and used in the first products of the next.
//     The last 12 products of the step hide them; what is left of their way is waited for with the next step's rows, at its end.
//     A wavefront follows the one with its number in the workgroup in front, which says so itself when its
//     stores have arrived, half a step after them: one flag a workgroup, behind the step's barrier, left the next one further behind and made it wait for the slowest
//     wavefront (64 units of 3000 tokens 904 us instead of 801, 48 of 8190 4210 instead of 4110).
//   * LDS, 149 KiB: K of the owners (B operand of S for their wavefront, A operand of dQ for all), two steps of Q and dO, three of dS.  dQ of two steps is formed at
//     once, so that each of the 8 wavefronts has a tile of 32 queries x 32 channels and all have the same work: half of the wavefronts each step, in turn,
//     left the others waiting at the barrier (5300 clocks a step instead of 4660).
//   * The initial logits and dP of the queries (-lse / scale, -delta) are formed by the launch in front, laid out as the steps read them, and come straight into LDS
//     like the rows: loaded into registers and multiplied there, wavefront 0 waited for them at the start of each step (6600 clocks instead of 5300).
//   * No spilled value is read in the walk: a scratch load waits for all loads in front of it, the next step's rows among them (133 ms with 50 spilled
//     values, 97 with 8).  Hence addresses are formed where they are used, and V's rows are registers and K's not.
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
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;

#define LDS_PTR(T) __attribute__((address_space(3))) T*

namespace {

constexpr int D = 128, KS = D / 16, MT = D / 32, CH = D / 8, RB = D * 2, RPI = 64 / CH;
constexpr int NW = 8, OWNERS = CHAIN_OWNERS, STEP = CHAIN_STEP;
static_assert(OWNERS == 32 * NW && STEP == 32 && NW * RPI == STEP, "a wavefront fetches one instruction of each streamed tensor a step");
constexpr int RING_AHEAD = 8, RING = 16;  // row offsets are formed this many groups of 64 rows ahead; groups kept in LDS
constexpr float LOG2E = 1.4426950408889634f;
constexpr int TILE = STEP * RB;         // bytes of a step's rows of one tensor
constexpr int DS_TILE = OWNERS * STEP * 2;
constexpr uint32_t MOST_TRIES = 1u << 22;  // of a wait for another workgroup, at about a microsecond each: no wait comes near it
constexpr int SC1 = 16;                    // cache policy of a buffer load: past the vector L1, which other CUs' stores do not reach

struct Lds {
    char *q0, *q1, *do0, *do1, *k, *ds;
    float *vals0, *vals1;  // initial S and dP per streamed row
    uint32_t* rowoff;
};

// The next (unit, block of keys) of this XCD.  Units are handed out a group at a time (BwdChain::task()).
// Every wait is for a workgroup that holds an earlier ticket of the same XCD: one that runs already, whose own waits are for still earlier ones.  A wait for the
// group's number that ran out all the same would drop the block: its dk and dv, and dq of a unit's last block, keep the NaN of the launch in front, and the block
// behind it finds no sums (see leave_sums).
__device__ inline uint32_t take_task(const BwdChain& w, uint32_t xcc) {
    const uint32_t n = __hip_atomic_fetch_add(w.ctl + xcc * 32u, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const uint32_t g = n / w.per_group, r = n - g * w.per_group;
    if (g > w.n_groups) return CHAIN_NONE;  // no XCD has more than all groups and one that was refused
    uint32_t* const slot = w.ctl + CHAIN_SLOTS + xcc * (w.n_units + 1u) + g;
    uint32_t id;
    if (r == 0u) {
        id = 1u + __hip_atomic_fetch_add(w.ctl + CHAIN_NEXT, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(slot, id, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    } else {
        uint32_t tries = 0;
        while ((id = __hip_atomic_load(slot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) == 0u && ++tries < MOST_TRIES) __builtin_amdgcn_s_sleep(1);
        if (id == 0u) return CHAIN_NONE;
    }
    return w.task(id, r);
}

template <bool PAD>
__device__ __attribute__((always_inline)) inline void chain_task(const BwdArgs& a, const PadArg<PAD>& pad_map, const BwdChain& w, const UnitMap& units, uint32_t lin, uint32_t tid, const Lds& lds) {
    uint32_t lane = tid & 63u;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t lq = lane & 31u, h = lane >> 5;
    const UnitAt at_unit = units.at<PAD>(lin);
    const uint32_t ot = at_unit.tile, bb = at_unit.bb, head = at_unit.head, p = at_unit.p, q = at_unit.q, b0 = at_unit.b;
    const ClassMap cm = make_class_map(a.g, pad_map, p, q);
    const uint32_t n_seq = PAD ? __builtin_amdgcn_readfirstlane(cm.n) : (uint32_t)a.g.n_sub;
    if (PAD && ot * (uint32_t)OWNERS >= n_seq) return;  // blocks are counted for the largest class
    const size_t C = (size_t)a.heads * D;
    const size_t unit_off = (size_t)b0 * (uint32_t)a.g.n_tok * C + (size_t)head * D;  // elements
    const float* const vals_u = w.vals + (size_t)(bb * (uint32_t)a.heads + head) * w.n_steps * (2 * STEP);
    const char* q_g = (const char*)((const __bf16*)a.q + unit_off);
    const char* do_g = (const char*)((const __bf16*)a.dout + unit_off);
    const bool first = ot == 0u, last = (ot + 1u) * (uint32_t)OWNERS >= n_seq;

    auto token_at = [&](uint32_t j) __attribute__((always_inline)) -> uint32_t {
        return PAD ? src_token_real(a.g, cm, p, q, j) : src_token(a.g, p, q, j);
    };
    const float c = a.scale * LOG2E;
    auto swz = [](uint32_t r) __attribute__((always_inline)) -> uint32_t { return lds_swizzle<D>(r); };

    // ---- streamed rows, as in attn_bwd.hip
    const uint32_t row_bytes = (uint32_t)C * 2u;
    const uint32_t n_t = (n_seq + STEP - 1) / STEP;
    auto produce = [&](uint32_t group) __attribute__((always_inline)) {
        const uint32_t j = group * 64u + lane;
        lds.rowoff[group % RING * 64u + lane] = token_at(j < n_seq ? j : n_seq - 1u) * row_bytes;
    };
    const uint32_t st_row = wave * RPI + lane / CH, st_cb = ((lane % CH) ^ swz(st_row)) * 16u;
    auto read_offs = [&](uint32_t t) __attribute__((always_inline)) -> uint32_t { return lds.rowoff[t * STEP % (RING * 64u) + st_row] + st_cb; };
    auto issue_tile = [&](uint32_t t, uint32_t off, char* b1, char* b2, float* vals) __attribute__((always_inline)) {
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(q_g + off), (LDS_PTR(void))(b1 + wave * 1024u), 16, 0, 0);
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(do_g + off), (LDS_PTR(void))(b2 + wave * 1024u), 16, 0, 0);
        if (wave == 0u) __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(vals_u + (size_t)t * (2 * STEP) + lane), (LDS_PTR(void))vals, 4, 0, 0);
    };
    auto landed = [&]() __attribute__((always_inline)) { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); };
    {
        const uint32_t j = lane & (uint32_t)(STEP - 1);
        const uint32_t mine = token_at(j < n_seq ? j : n_seq - 1u) * row_bytes;
        issue_tile(0, (uint32_t)__shfl((int)mine, (int)st_row) + st_cb, lds.q0, lds.do0, lds.vals0);
    }

    // ---- owners: K rows in LDS for all wavefronts (B operand of S for their wavefront, A operand of dQ for all), V rows in registers
    const uint32_t jo = ot * (uint32_t)OWNERS + wave * 32u + lq;
    const uint32_t own_tok = token_at(jo < n_seq ? jo : n_seq - 1u);
    {
        const char* k_g = (const char*)((const __bf16*)a.k + unit_off);
#pragma unroll
        for (int i = 0; i < 32 / RPI; i++) {
            const uint32_t r = i * RPI + lane / CH;
            const uint32_t off = (uint32_t)__shfl((int)own_tok, (int)r) * row_bytes + (((lane % CH) ^ swz(r)) * 16u);
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(k_g + off), (LDS_PTR(void))(lds.k + wave * 32u * RB + i * 1024u), 16, 0, 0);
        }
    }
    bf16x8 own_v[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ks++) own_v[ks] = *(const bf16x8*)((const __bf16*)a.v + unit_off + (size_t)own_tok * C + ks * 16 + 8 * h);
    const float own_off = jo < n_seq ? 0.f : -INFINITY;  // an owner past the end has P = 0: it must not add to dQ

    f32x16 dk[MT], dv[MT];
#pragma unroll
    for (int mt = 0; mt < MT; mt++)
#pragma unroll
        for (int r = 0; r < 16; r++) dk[mt][r] = dv[mt][r] = 0.f;

    // ---- read addresses
    uint32_t a_rd0 = lq * RB + ((h ^ swz(lq)) * 16u);
    auto a_rd = [&](int ks) __attribute__((always_inline)) -> uint32_t { return a_rd0 ^ (uint32_t)(ks * 32); };
    const char* const own_k = lds.k + wave * 32u * RB;
    const uint32_t li = lane & 15u, lgrp = (lane >> 4) & 1u;
    uint32_t t_rd[2];  // channel block 0; block mt has mt * 64 XORed in
#pragma unroll
    for (int sec = 0; sec < 2; sec++) {
        const uint32_t row = 4 * h + (li >> 2) + 8 * sec, ch = lgrp * 2 + ((li & 3u) >> 1);
        t_rd[sec] = row * RB + ((ch ^ swz(row)) * 16u) + 8 * (li & 1u);
    }
    // dS of a step: [key][query], 64 bytes a key, chunk (8 queries) c of key k at position c ^ (k/4 % 4): neither the 8-byte writes (32 keys) nor the transposing
    // reads (8 keys x 32 queries) meet in a bank
    uint32_t ds_wr = (wave * 32u + lq) * 64u + h * 8u, ds_sw = (lq >> 2 & 3u) * 16u;
    uint32_t ds_rd[2];
#pragma unroll
    for (int sec = 0; sec < 2; sec++) {
        const uint32_t key = 4 * h + (li >> 2) + 8 * sec, ch = lgrp * 2 + ((li & 3u) >> 1);
        ds_rd[sec] = key * 64u + ((ch ^ (key >> 2 & 3u)) * 16u) + 8 * (li & 1u);
    }

    // ---- the chain: sums of step t of this unit, 16 KiB: [channel block][register / 4][lane][4]
    const uint32_t cb = wave & 3u, half = wave >> 2;
    float* const part_u = w.part + (size_t)at_unit.unit * w.n_steps * (STEP * D);
    uint32_t* const done = w.ctl + CHAIN_SLOTS + CHAIN_XCCS * (w.n_units + 1u) + lin * CHAIN_FLAGS + wave;  // steps that this wavefront has left; [-CHAIN_FLAGS]: that of the workgroup before
    uint32_t seen = 0;
    bool lost = false;
    auto wait_for = [&](uint32_t steps) __attribute__((always_inline)) {
        uint32_t have = __builtin_amdgcn_readfirstlane(seen), tries = 0;
#pragma unroll 1
        while (have < steps && !lost) {
            __builtin_amdgcn_s_sleep(1);
            seen = __hip_atomic_load(done - CHAIN_FLAGS, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            have = __builtin_amdgcn_readfirstlane(seen);
            lost = ++tries >= MOST_TRIES;
        }
        asm volatile("" ::: "memory");
    };
    auto part_rsrc = [&](uint32_t t) __attribute__((always_inline)) {
        return __builtin_amdgcn_make_buffer_rsrc(part_u + (size_t)t * (STEP * D) + cb * (32u * 32u), 0, 4096, 0x00020000);
    };
    // dQ^T[channel, query] += K^T dS^T over the 256 keys, 16 a product
    auto add_products = [&](const char* ds, f32x16& x) __attribute__((always_inline)) {
        constexpr int AH = 3;
        bf16x8 fk[16], fs[16];
        const uint32_t x0 = t_rd[0] ^ (cb * 64u), x1 = t_rd[1] ^ (cb * 64u);
        auto read = [&](int s) __attribute__((always_inline)) {
            const bf16x4 k0 = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((LDS_PTR(bf16x4))(LDS_PTR(char))(lds.k + x0 + s * 16 * RB));
            const bf16x4 k1 = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((LDS_PTR(bf16x4))(LDS_PTR(char))(lds.k + x1 + s * 16 * RB));
            const bf16x4 d0 = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((LDS_PTR(bf16x4))(LDS_PTR(char))(ds + ds_rd[0] + s * 16 * 64));
            const bf16x4 d1 = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((LDS_PTR(bf16x4))(LDS_PTR(char))(ds + ds_rd[1] + s * 16 * 64));
            fk[s] = __builtin_shufflevector(k0, k1, 0, 1, 2, 3, 4, 5, 6, 7);
            fs[s] = __builtin_shufflevector(d0, d1, 0, 1, 2, 3, 4, 5, 6, 7);
        };
#pragma unroll
        for (int s = 0; s < AH; s++) read(s);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int s = 0; s < 16; s++) {
            if (s + AH < 16) read(s + AH);
            x = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fk[s], fs[s], x, 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    auto leave_sums = [&](uint32_t t, f32x16& x) __attribute__((always_inline)) {
        if (lost) x[0] = __builtin_nanf("");  // no wait for the workgroup in front ends so; if one did, dq would say it
        if (!last) {
            const auto rsrc = part_rsrc(t);
#pragma unroll
            for (int g = 0; g < 4; g++) {
                const f32x4 v = {x[4 * g], x[4 * g + 1], x[4 * g + 2], x[4 * g + 3]};
                __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), rsrc, (int)(lane * 16u), g * 1024, 0);
            }
            return;
        }
        // lane = query lq; its row's offset is still in the ring
        if (t * STEP + lq < n_seq) {
            char* const at = (char*)((__bf16*)a.dq + unit_off) + lds.rowoff[(t * STEP + lq) % (RING * 64u)] + cb * 64u + h * 8u;
#pragma unroll
            for (int g = 0; g < 4; g++) {
                bf16x4 o;
#pragma unroll
                for (int e = 0; e < 4; e++) o[e] = (__bf16)(x[4 * g + e] * a.scale);
                *(bf16x4*)(at + g * 16) = o;
            }
        }
    };

    for (uint32_t g = wave; g < (uint32_t)RING_AHEAD; g += NW) produce(g);
    landed();
    __syncthreads();
    uint32_t off_next = read_offs(1);

    f32x16 x;
    auto take_sums = [&](uint32_t t, uint32_t steps) __attribute__((always_inline)) {
        if (first) {
#pragma unroll
            for (int r = 0; r < 16; r++) x[r] = 0.f;
            return;
        }
        wait_for(steps);
        const auto rsrc = part_rsrc(t);
#pragma unroll
        for (int g = 0; g < 4; g++) {
            const f32x4 v = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)(lane * 16u), g * 1024, SC1));
#pragma unroll
            for (int e = 0; e < 4; e++) x[4 * g + e] = v[e];
        }
    };
    auto pass_on = [&](uint32_t t, const char* ds) __attribute__((always_inline)) {
        add_products(ds, x);
        leave_sums(t, x);
    };
    // Step t: products of queries t.  Before an even one all wavefronts form dQ of the two steps before it, whose dS all have left in LDS: each 32 channels of
    // the queries of one of them.
    uint32_t ds_at = 0;  // of step t
    auto ds_ahead = [](uint32_t at) __attribute__((always_inline)) -> uint32_t { return at == 2u * DS_TILE ? 0u : at + DS_TILE; };
    auto ds_behind = [](uint32_t at) __attribute__((always_inline)) -> uint32_t { return at == 0u ? 2u * DS_TILE : at - DS_TILE; };
    auto do_step = [&](auto PARC, uint32_t t) __attribute__((always_inline)) {
        constexpr int PARITY = decltype(PARC)::value;  // t & 1
        const bool more = t + 1u < n_t;
        const char* t1 = PARITY ? lds.q1 : lds.q0;
        const char* t2 = PARITY ? lds.do1 : lds.do0;
        char* const ds_now = lds.ds + ds_at;
        // addresses are formed from these where they are used: kept in registers through the walk they do not fit
        asm volatile("" : "+v"(a_rd0), "+v"(t_rd[0]), "+v"(t_rd[1]), "+v"(ds_wr), "+v"(ds_sw), "+v"(lane));
        const uint32_t off_now = off_next;
        off_next = read_offs(t + 2u);
        if (PARITY == 0 && wave == (t / 2u & (uint32_t)(NW - 1))) produce(t / 2u + RING_AHEAD);
        if (more) issue_tile(t + 1u, off_now, PARITY ? lds.q0 : lds.q1, PARITY ? lds.do0 : lds.do1, PARITY ? lds.vals0 : lds.vals1);
        if ((PARITY == 1 || !more) && !first) seen = __hip_atomic_load(done - CHAIN_FLAGS, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (PARITY == 0 && t != 0u) pass_on(t - 2u + half, lds.ds + (half ? ds_behind(ds_at) : ds_ahead(ds_at)));
        f32x16 m1, m2;
#pragma unroll
        for (int g = 0; g < 4; g++) {
            const f32x4 i1 = *(const f32x4*)&(PARITY ? lds.vals1 : lds.vals0)[8 * g + 4 * h];
            const f32x4 i2 = *(const f32x4*)&(PARITY ? lds.vals1 : lds.vals0)[STEP + 8 * g + 4 * h];
#pragma unroll
            for (int e = 0; e < 4; e++) {
                m1[4 * g + e] = i1[e];
                m2[4 * g + e] = i2[e];
            }
        }
        // S, then dP; the exponentials of S are issued between the products of dP, and dS is formed between those of dV, which need P alone.  Every fragment is
        // read AH products before its own, and the order is pinned.
        constexpr int AH_A = 3, AH_C = 2;
        bf16x8 fa[2 * KS], ka[KS];
        auto read_a = [&](int g) __attribute__((always_inline)) {
            fa[g] = *(const bf16x8*)((g < KS ? t1 : t2) + a_rd(g % KS));
            if (g < KS) ka[g] = *(const bf16x8*)(own_k + a_rd(g));
        };
        auto frag_c = [&](int cidx) __attribute__((always_inline)) -> bf16x8 {
            const int g2 = cidx / MT % 2, mt = cidx % MT;
            const char* ta = (cidx < 2 * MT ? t2 : t1) + g2 * 16 * RB;
            const bf16x4 v0 = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((LDS_PTR(bf16x4))(LDS_PTR(char))(ta + (t_rd[0] ^ (uint32_t)(mt * 64))));
            const bf16x4 v1 = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((LDS_PTR(bf16x4))(LDS_PTR(char))(ta + (t_rd[1] ^ (uint32_t)(mt * 64))));
            return __builtin_shufflevector(v0, v1, 0, 1, 2, 3, 4, 5, 6, 7);
        };
        bf16x8 rf[2], rp[2], fc[4 * MT];
#pragma unroll
        for (int g = 0; g < AH_A; g++) read_a(g);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int g = 0; g < KS; g++) {
            read_a(g + AH_A);
            m1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[g], ka[g], m1, 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int g = KS; g < 2 * KS; g++) {
            if (g + AH_A < 2 * KS) read_a(g + AH_A);
            else if (g + AH_C >= 2 * KS) fc[g + AH_C - 2 * KS] = frag_c(g + AH_C - 2 * KS);
            m2 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[g], own_v[g - KS], m2, 0, 0, 0);
            const int r = 2 * (g - KS);
            f32x2 prob;
#pragma unroll
            for (int u = 0; u < 2; u++) m1[r + u] = prob[u] = __builtin_amdgcn_exp2f(fmaf(m1[r + u], c, own_off));
            const bf16x2 pb = __builtin_convertvector(prob, bf16x2);
            rp[r / 8][r % 8] = pb[0];
            rp[r / 8][r % 8 + 1] = pb[1];
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int cidx = 0; cidx < 4 * MT; cidx++) {
            const int g2 = cidx / MT % 2, mt = cidx % MT;
            if (cidx + AH_C < 4 * MT) fc[cidx + AH_C] = frag_c(cidx + AH_C);
            if (cidx < 2 * MT) {
                dv[mt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fc[cidx], rp[g2], dv[mt], 0, 0, 0);
                const int r = 2 * cidx;
                const f32x2 val = {m1[r] * m2[r], m1[r + 1] * m2[r + 1]};
                const bf16x2 vb = __builtin_convertvector(val, bf16x2);
                rf[r / 8][r % 8] = vb[0];
                rf[r / 8][r % 8 + 1] = vb[1];
                if (cidx % 2 == 1) {
                    const int k = cidx / 2;  // queries 8k + 4h ..
                    *(bf16x4*)(ds_now + ds_wr + ((uint32_t)k * 16u ^ ds_sw)) = k % 2 == 0 ? __builtin_shufflevector(rf[k / 2], rf[k / 2], 0, 1, 2, 3) : __builtin_shufflevector(rf[k / 2], rf[k / 2], 4, 5, 6, 7);
                }
            } else {
                dk[mt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fc[cidx], rf[g2], dk[mt], 0, 0, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
            if (cidx == MT - 1) {
                if (PARITY == 0 && t != 0u) {
                    landed();  // the sums that this wavefront has left, half a step ago
                    if (lane == 0u) __hip_atomic_store(done, t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
                asm volatile("" : "=v"(x));  // not the sums that have left
                if (PARITY == 1) take_sums(t - 1u + half, t + 1u);
                else if (!more && half == 0u) take_sums(t, t + 1u);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        landed();  // the next step's rows
        __syncthreads();
        ds_at = ds_ahead(ds_at);
    };
    using P0 = std::integral_constant<int, 0>;
    using P1 = std::integral_constant<int, 1>;
    uint32_t t = 0;
    for (; t + 1 < n_t; t += 2) {
        do_step(P0{}, t);
        do_step(P1{}, t + 1u);
    }
    if (t < n_t) do_step(P0{}, t);
    // dQ of the last two steps, or of the last one
    if (n_t & 1u) {
        if (half == 0u) pass_on(n_t - 1u, lds.ds + ds_behind(ds_at));
    } else {
        pass_on(n_t - 2u + half, lds.ds + (half ? ds_behind(ds_at) : ds_ahead(ds_at)));
    }
    landed();
    if (lane == 0u) __hip_atomic_store(done, n_t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();

    const uint32_t stored = rows_below(ot * (uint32_t)OWNERS + wave * 32u, n_seq);
    if (stored == 0u) return;
    const uint32_t in = wave / 2u;
    char* const region = (in == 0 ? lds.q0 : in == 1 ? lds.q1 : in == 2 ? lds.do0 : lds.do1) + wave % 2u * 4096u;
    const RowDest<64> dest(own_tok, C, stored, lane);
    store_rows<64, 32>(region, dk, a.scale, (__bf16*)a.dk + unit_off, dest, lane);
    store_rows<64, 32>(region, dv, 1.0f, (__bf16*)a.dv + unit_off, dest, lane);
}

// As many workgroups as the chip has CUs, each taking tasks until there are none.  Which of them do what does not matter for the result.
template <bool PAD>
__global__ __launch_bounds__(64 * NW, 1) void attn_bwd_chain_kernel(BwdArgs a, PadArg<PAD> pad_map, UnitMap units, BwdChain w) {
    __shared__ __attribute__((aligned(1024))) char q0[TILE], q1[TILE], do0[TILE], do1[TILE], k[OWNERS * RB], ds[3 * DS_TILE];
    __shared__ __attribute__((aligned(16))) float vals0[2 * STEP], vals1[2 * STEP];
    __shared__ __attribute__((aligned(16))) uint32_t rowoff[RING * 64];
    __shared__ uint32_t task;
    const uint32_t xcc = __builtin_amdgcn_s_getreg(20 | 0 << 6 | 3 << 11);  // HW_REG_XCC_ID, 4 bits
    for (;;) {
        uint32_t tid = threadIdx.x;
        asm volatile("" : "+v"(tid));  // formed anew for each task: nothing of a walk is kept in registers over the next
        __syncthreads();  // the task before this one has read its LDS
        if (tid == 0u) task = take_task(w, xcc);
        __syncthreads();
        const uint32_t lin = __builtin_amdgcn_readfirstlane(task);
        if (lin == CHAIN_NONE) return;
        if (lin == CHAIN_SKIP) continue;
        chain_task<PAD>(a, pad_map, w, units, lin, tid, {q0, q1, do0, do1, k, ds, vals0, vals1, rowoff});
    }
}

template <bool PAD>
hipError_t launch_t(const BwdArgs& a, const BwdChain& w, hipStream_t stream) {
    PadArg<PAD> pad_map;
    make_pad_arg(a.g, pad_map);
    const uint64_t tasks = (uint64_t)w.n_units * w.n_blk;
    attn_bwd_chain_kernel<PAD><<<(uint32_t)(tasks < CUS ? tasks : CUS), 64 * NW, 0, stream>>>(a, pad_map, make_unit_map<PAD>(a.g, w.n_blk, (uint32_t)a.B, (uint32_t)a.heads), w);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_attn_bwd_chain(const BwdArgs& a, const BwdChain& w, hipStream_t stream) {
    const hipError_t e = launch_bwd_chain_start(a, w, stream);
    if (e != hipSuccess) return e;
    return a.pad ? launch_t<true>(a, w, stream) : launch_t<false>(a, w, stream);
}

}  // namespace skiparse

// Which workgroup shape an attention launch gets.  A kernel exists in a few shapes that differ in the rows (queries, or keys in the
// dK+dV launch) a workgroup takes and in whether two groups of wavefronts share the walk over the other side; large workgroups move the
// least data per MFMA, small ones fill the chip when the problem is small.
#pragma once
#include <stdint.h>

namespace skiparse {

struct ShapeCost {
    int shape;       // FwdShape or BwdShape
    int rows;        // rows of a workgroup
    bool split;      // two groups that walk half of the rows each
    int max_k;       // workgroups of this shape that one CU holds
    float first;     // us outside the walk (prologue, pipeline fill, epilogue, merge): the first round of workgroups,
    float again;     // and every further one
    float crowd;     // once, where workgroups share a CU: they start together and wait for the same loads
    float block[4];  // us per 32-row block of the walk with 128 or fewer, 256, 512, 768 workgroups running
    // how much of the difference to a full round a last round of many has, from the round's half on: the chip's clock is down by then, and its workgroups begin
    // here and there, as the others end (without it the fit took 69x1304 to Q256, 82 us instead of 72)
    float late = 0.f;
};

// The units of a launch: how many have any row, and the rows of the largest and of the smallest one (they differ in the any-resolution
// mode only).
struct UnitSizes {
    uint64_t units;
    uint32_t n_max, n_min;
    uint64_t workgroups(const ShapeCost& c) const { return units * ((n_max + (uint32_t)c.rows - 1u) / (uint32_t)c.rows); }
};

constexpr uint64_t CUS = 256;
constexpr uint32_t GROUP_MIN_ROWS = 64;  // a group of wavefronts needs a tile of its own: units of this size or less are not split

// us per block with `wgs` workgroups running: between the entries the cost is linear (the chip's clock falls as it fills, and CUs with two
// workgroups slow down by and by), or with `step` that of the entry above.
inline float block_cost(const ShapeCost& c, uint64_t wgs, bool step) {
    const int hi = wgs <= CUS ? 1 : (int)((wgs - 1u) / CUS) + 1;
    if (step) return c.block[hi];
    if (wgs <= CUS / 2) return c.block[0];
    const float from = hi == 1 ? CUS / 2 : (float)(CUS * (hi - 1)), width = hi == 1 ? CUS / 2 : CUS;
    return c.block[hi - 1] + (c.block[hi] - c.block[hi - 1]) * ((float)wgs - from) / width;
}

// Estimated us of a launch: rounds over the CUs, the last one with what is left.
inline float launch_cost(const ShapeCost& c, const UnitSizes& u, bool step) {
    const float blocks = (float)((u.n_max + 31u) / 32u);
    const uint64_t wgs = u.workgroups(c), per_round = CUS * (uint64_t)c.max_k, rounds = wgs / per_round, rem = wgs % per_round;
    float t = c.first + c.again * (float)(rounds + (rem != 0) - 1u) + (float)rounds * blocks * c.block[c.max_k];
    if (rem != 0) {
        float b = block_cost(c, rem, step);
        if (rounds != 0) b += c.late * (2u * rem < per_round ? 2.0f * (float)rem / (float)per_round : 1.0f) * (c.block[c.max_k] - b);
        t += blocks * b;
    }
    if (wgs > CUS) t += c.crowd * (wgs >= CUS + CUS / 12 ? 1.0f : 12.0f * (float)(wgs - CUS) / CUS);
    return t;
}

// The shape with the smallest estimate among those that `admit` lets through; the first one always is.
template <int N, typename Admit>
inline int pick_shape(const ShapeCost (&cost)[N], const UnitSizes& u, bool step, Admit admit) {
    int best = 0;
    float best_t = launch_cost(cost[0], u, step);
    for (int v = 1; v < N; v++) {
        if ((cost[v].split && u.n_min <= GROUP_MIN_ROWS) || !admit(cost[v])) continue;
        const float t = launch_cost(cost[v], u, step);
        if (t < best_t) {
            best = v;
            best_t = t;
        }
    }
    return cost[best].shape;
}

// ---- forward
enum FwdShape : int {
    Q256 = 1,        // 8 wavefronts, 1 group: 256 queries share every tile; the least L2 -> LDS traffic per MFMA, the best once the chip is full
    Q128 = 2,        // 4 wavefronts, 1 group: two (head_dim 64: three) workgroups per CU; twice as many, finer-grained workgroups
    Q64_SPLIT = 3,   // 4 wavefronts, 2 groups: four times the workgroups, half the serial chain
    Q128_SPLIT = 4,  // 8 wavefronts, 2 groups: half the chain at two wavefronts per SIMD
    // Q256 and Q128 for units whose wavefronts all have a query: see fwd_kernel()
    Q256_FULL = 5,
    Q128_FULL = 6,
};

// Costs fitted to 1200 calls timed in every shape, in turn and warm (1..640 units of 16..12,000 tokens), and held to the calls named below: the pick is 0.07 % above
// the best shape on average at head_dim 128 (6 % at worst) and 0.04 % at head_dim 64 (5 %).  Against the fit to the kernels that stored their results in pieces,
// whose ends and merges took longer, 0.978 and 0.985 of the time on average (0.84 at best; at worst 1.004, 10x1512 and 4x3293, and 1.044, 63x1574 at head_dim 64, which
// moved from Q128 to Q256: 65.5 us against 62.7).  Q64_SPLIT at
// head_dim 64 has become 8 to 12 % faster since (fwd_per_cu() in attn_fwd.hip), and its row is fitted to 1000 calls timed anew: 0.24 % above the best on average and 11 %
// at worst, where the old one was 0.54 and 30 % (3x5414 50.4 us in Q128_SPLIT, 41.6 in Q64_SPLIT).  Measured, us, Q256 / Q128 / Q64_SPLIT /
// Q128_SPLIT at head_dim 128, units x tokens: 78x67 6.30 / 6.11 / 7.31 / 7.11, 10x1512 36.1 / 27.9 / 23.8 / 23.9, 69x1304 82.3 / 72.4 / 133 / 79.7, 4x3293 71.6 / 55.1 /
// 43.7 / 43.9; 192x240, 34x900, 84x512, 48x960, 14x30240 and 20x20160 keep Q256.  At head_dim 64: 52x276 8.47 / 6.87 / 8.38 / 7.19, 10x3203 57 / 57 / 44 / 62, 100x4096
// and 160x20160 keep Q128; 103x377 keeps Q256.
//   * What a round costs depends on how full it is: a Q256 block takes 0.74 us with half of the CUs busy and 0.97 with all of them, the chip
//     being at its power limit.  Without that the rule gave long sequences to Q128_SPLIT for a smaller last round.
//   * Two Q128 workgroups that start together on a CU wait for the same loads (`crowd`).
//   * Q64_SPLIT is for one round of its own: in a second one the traffic of four times the workgroups shows.
//     (The earlier kernels, Q256 / the other one: 14x30240 5740 / 6025, 192x240 16.5 / 17.3, 84x512 21.3 / 22.5, 34x900 29 / 33.5.)
//   * The split shapes stream K and V at two places and move 4 % more per MFMA; what they gain is idle CUs, so they are left out from two
//     rounds of Q256 on.
constexpr ShapeCost FWD_COST_128[] = {{Q256, 256, false, 1, 4.43f, 6.52f, 0.f, {0.742f, 0.967f}, 0.65f},
                                      {Q128, 128, false, 2, 4.11f, 2.15f, 1.84f, {0.443f, 0.775f, 1.051f}, 0.20f},
                                      {Q64_SPLIT, 64, true, 1, 5.62f, 1.49f, 0.f, {0.305f, 0.347f}},
                                      {Q128_SPLIT, 128, true, 1, 6.50f, 14.55f, 0.f, {0.319f, 0.548f}}};
constexpr ShapeCost FWD_COST_64[] = {{Q256, 256, false, 1, 2.44f, 6.90f, 0.f, {0.310f, 0.528f}},
                                     {Q128, 128, false, 3, 1.01f, 1.87f, 4.97f, {0.320f, 0.346f, 0.514f, 0.658f}},
                                     {Q64_SPLIT, 64, true, 2, 2.32f, 0.48f, 0.56f, {0.095f, 0.179f, 0.282f}},
                                     {Q128_SPLIT, 128, true, 1, 2.38f, 9.52f, 0.f, {0.179f, 0.251f}}};
inline int pick_fwd_shape(int head_dim, const UnitSizes& u) {
    const auto& cost = head_dim == 128 ? FWD_COST_128 : FWD_COST_64;
    return pick_shape(cost, u, false, [&](const ShapeCost& c) {
        if (!c.split) return true;
        return u.workgroups(cost[0]) < 2u * CUS && (c.shape != Q64_SPLIT || u.workgroups(c) <= CUS * (uint64_t)c.max_k);
    });
}

// The kernel of a launch.  The wavefronts past a unit's last query leave the arithmetic out; launches of the large shapes that have no such wavefront take
// the FULL kernels, without the test for it (in the any-resolution mode units differ in size, and nearly all launches have some), and so does Q64_SPLIT at
// head_dim 128, where it cost 0.3 to 1.2 % whatever the size.  Over 240 random calls, without -> with the test, us: 320 units of 540 tokens at head_dim 64
// 44.8 -> 42.7, 422 of 32 4.55 -> 4.19, at head_dim 128 160 of 960 93.0 -> 90.6, 160 of 1440 185 -> 181; where every wavefront has a query 0.995 to 1.012
// of the time (40 of 384 at head_dim 64 6.97 -> 7.04); Q64_SPLIT at head_dim 128 3 of 440 10.26 -> 10.37, 25 of 260 9.20 -> 9.25; the other shapes of two
// groups 0.99 to 1.003; the any-resolution mode 0.93 to 1.009, the latter where few wavefronts are idle (68 units of 240 and 300 at head_dim 64).
// At head_dim 64, three workgroups a CU, it is FULL in more than one round as well if a unit is a multiple of 16 workgroups: the short ones meet on the
// same CUs (32 an XCD, in turn), which then take more than their share of the last round (40 of 4032 182 -> 189, 80 of 1984 94 -> 97).
inline int fwd_kernel(int head_dim, bool pad, const UnitSizes& u) {
    const int shape = pick_fwd_shape(head_dim, u);
    if (pad || (shape != Q256 && shape != Q128)) return shape;
    const uint32_t rows = shape == Q256 ? 256u : 128u, left = u.n_max % rows, per_unit = (u.n_max + rows - 1u) / rows;
    const bool idle = left != 0 && left + 32u <= rows;
    const bool meet = head_dim == 64 && shape == Q128 && per_unit % 16u == 0 && u.units * per_unit > 3u * CUS;
    return idle && !meet ? shape : shape == Q256 ? Q256_FULL : Q128_FULL;
}

// ---- backward.  The dQ owners are queries, the dK+dV owners keys.
enum BwdShape : int {
    // a launch of each kind of owner, 256 a workgroup (8 wavefronts), the dQ launch forming delta;
    TWO_LAUNCHES = 0,
    // or both kinds in ONE launch (after a small one that forms delta): the dK+dV workgroups first, the dQ workgroups fill the chip behind them, so that there
    // is one last round instead of two and a call of few units has twice the workgroups
    B128 = 1,        // 4 wavefronts, 1 group, two workgroups on a CU whatever their kind
    B64_SPLIT = 2,   // 4 wavefronts, 2 groups
    B128_SPLIT = 3,  // 8 wavefronts, 2 groups
    // as TWO_LAUNCHES, with 128 queries (4 wavefronts) a workgroup in the dQ launch
    TWO_LAUNCHES_DQ128 = 4,
};

// us, the mean of both kinds.  Fitted to 660 calls (1..1088 units of 24..30,000 tokens, plain and any-resolution) timed in every shape: the pick is 0.5 %
// above the best on average and 12 % at worst, and 0.84 of the two launches' time on average (1.03 at worst).  Measured, two launches -> picked,
// us, units x tokens, head_dim 128: 1x120 18.1 -> 12.4, 8x190 21.6 -> 14.5, 48x400 43 -> 35, 24x1000 75 -> 63.5, 1x6116 215 -> 134, 160x400 120 -> 93,
// 160x960 344 -> 312, 1x11191 390 -> 370, 12x8190 1437 -> 1313, 4x20160 3387 -> 2704, 160x2600 2093 -> 1977; head_dim 64: 1x78 11.8 -> 8.1,
// 48x400 25.9 -> 21.4, 24x1000 44.6 -> 33.8, 1x3955 94 -> 52, 4x5000 171 -> 115, 160x960 171 -> 165.
// The ends and merges of the workgroups have become shorter since, by about the same for all, so that the picks stand (0.3 % above the best on average over 900
// calls timed anew); units of 65 to 96 tokens at head_dim 128 alone are better off in B128 than in two groups (7x74 12.1 -> 10.4 us): `first` of B64_SPLIT.
constexpr ShapeCost PAIR_COST_128[] = {{B128, 128, false, 2, 8.9f, 8.3f, 4.7f, {1.285f, 1.505f, 1.616f}},
                                       {B64_SPLIT, 64, true, 1, 11.2f, 4.0f, 0.f, {0.614f, 0.718f}},
                                       {B128_SPLIT, 128, true, 1, 14.3f, 8.2f, 0.f, {0.975f, 0.930f}}};
constexpr ShapeCost PAIR_COST_64[] = {{B128, 128, false, 2, 7.2f, 5.4f, 2.4f, {0.558f, 0.684f, 0.848f}},
                                      {B64_SPLIT, 64, true, 2, 7.4f, 4.0f, 1.8f, {0.361f, 0.387f, 0.481f}},
                                      {B128_SPLIT, 128, true, 1, 11.6f, 6.1f, 0.f, {0.372f, 0.426f}}};
// Workgroups of 256 owners, in a launch of each kind, take 4 to 7 % less per row and block (head_dim 64: 1 to 4 %), but only their full rounds show
// it: the share of the chip's rounds that holds owners has to be near one, or there is a single, largely filled round of a long walk.  (At head_dim 128 the larger ones
// come here on the least workspace only: bwd_chain().)  Measured, one launch
// in B128 -> two of 256 owners, us: 73x12282 1.00 -> 0.932, 192x4584 0.953, 48x8190 5295 -> 5081, 84x3740 2026 -> 1918, 582x2734 7870 -> 7700, 160x20160 105,350 -> 102,340, 6x7844 (162 workgroups)
// 0.900; the other way 20x20160 13,570 -> 13,940, 39x5781 1.011, 414x1824 1.058, 74x385 1.246.
inline bool bwd_full_rounds(int head_dim, const UnitSizes& u) {
    const uint64_t wgs = u.units * ((u.n_max + 255u) / 256u), rounds = (wgs + CUS - 1u) / CUS;
    const float fill = (float)(u.units * ((u.n_max + 127u) / 128u)) / (float)(2u * CUS * rounds);
    // Classes of different sizes and many rounds (head_dim 128): the two launches stay 1 to 4 % ahead (972 units of 1596 to 2100 tokens 6530 -> 6340, 320 of
    // 5000 tokens 15,155 -> 14,780), where equal units gain up to 7 % by the one.
    if (head_dim == 128 && u.n_min != u.n_max && u.n_max >= 1500u && u.units * ((u.n_max + 127u) / 128u) >= 8u * CUS) return true;
    if (rounds == 1u) return head_dim == 128 ? u.n_max >= 2300u && fill >= 0.70f : u.n_max >= 1600u && fill >= 0.78f;
    if (head_dim == 128) return fill >= 0.955f ? u.n_max >= 2500u : u.n_max >= 4000u && fill >= 0.935f;
    return u.n_max >= 4000u && rounds <= 6u && fill >= 0.955f;
}

// Which dQ launch, where there are two: 128 queries a workgroup, two on a CU, have the better last round in some calls (24 units of 2055 tokens at head_dim 64).
// One figure for a round, however full, is enough here.
constexpr ShapeCost DQ_COST_128[] = {{TWO_LAUNCHES, 256, false, 1, 5.0f, 5.0f, 0.f, {0.f, 1.30f}}, {TWO_LAUNCHES_DQ128, 128, false, 2, 4.0f, 4.0f, 0.f, {0.f, 0.95f, 1.34f}}};
constexpr ShapeCost DQ_COST_64[] = {{TWO_LAUNCHES, 256, false, 1, 3.5f, 3.5f, 0.f, {0.f, 0.80f}}, {TWO_LAUNCHES_DQ128, 128, false, 2, 2.8f, 2.8f, 0.f, {0.f, 0.56f, 0.81f}}};
inline int pick_bwd_shape(int head_dim, const UnitSizes& u) {
    if (bwd_full_rounds(head_dim, u)) return pick_shape(head_dim == 128 ? DQ_COST_128 : DQ_COST_64, u, true, [](const ShapeCost&) { return true; });
    const UnitSizes both = {2u * u.units, u.n_max, u.n_min};
    // more rounds of the split shapes than these were never the best
    return pick_shape(head_dim == 128 ? PAIR_COST_128 : PAIR_COST_64, both, false, [&](const ShapeCost& c) {
        const uint64_t most = c.shape == B64_SPLIT ? (head_dim == 128 ? 1u : 3u) : c.shape == B128_SPLIT ? (head_dim == 128 ? 2u : 4u) : ~0u;
        return both.workgroups(c) <= most * CUS * (uint64_t)c.max_k;
    });
}

// ---- all gradients in one walk, dQ passed along a unit's workgroups (attn_bwd_chain.hip)
constexpr uint32_t XCDS = 8, CHAIN_OWNERS = 256, CHAIN_STEP = 32;  // keys of a workgroup, queries of a step
// Units handed to an XCD at a time, whose workgroups take turns on its CUs.  One unit makes a chain of 32 workgroups, each of which starts behind the one before it
// and waits where that one was late; of several less is found in the L2, which long walks pay for.  us, by 1 / 2 / 4, units x tokens: 64x3000 830 / 810 / 776,
// 160x4200 3964 / 3965 / 3887, 160x6000 7609 / 7642 / 7619, 48x8190 4221 / 4152 / 5239 (6 units an XCD), 64x12000 12,359 / 11,958 / 12,226, 160x12000 29,202 / 29,180 /
// 30,213, 32x20160 16,521 / 17,005 / 16,963, 160x20160 82,409 / 83,608 / 84,902.  The upper line rests on
// the last three sizes alone and lies somewhere between 12,000 tokens, where one and two are equal, and 20,160.  Never so many that the busiest XCD has more units than by one.
inline uint32_t chain_together(uint64_t units, uint32_t n_max) {
    const uint64_t least = (units + XCDS - 1u) / XCDS;
    for (uint32_t n = n_max >= 16000u ? 1u : n_max >= 7000u ? 2u : 4u; n > 1u; n--)
        if (((units + n - 1u) / n + XCDS - 1u) / XCDS * n == least) return n;
    return 1u;
}
// An XCD's CUs take its units' workgroups in rounds.  Two rounds or more that are largely filled take 0.82 to 0.98 of the time of the shapes above; chains of 32
// workgroups want longer walks.  Measured at 200 sizes, units x tokens: 160x20160 98.2 -> 80.6 ms, 48x8190 4817 -> 4092 us (0.85 and 0.88 of the time since the two
// launches have gained as well: 95.1 ms, 4650), 480x960 (0.88 full) 0.89 of the time,
// 64x2907 0.87, 48x4200 (0.77) 0.95, 64x2315 (0.75) 0.96; the other way 12x8116 (0.74) 1.09, 48x3000 (0.73) 1.03, 160x1017 (0.83) 1.02, 20x20160 (0.77, chains of 32)
// 1.04, 40x3000 (0.92, chains of 32) 1.13, 24x2343 (one round) 1.03.
inline bool bwd_chain(int head_dim, const UnitSizes& u) {
    if (head_dim != 128 || u.units == 0) return false;
    const uint64_t rounds = ((u.units + XCDS - 1u) / XCDS * ((u.n_max + CHAIN_OWNERS - 1u) / CHAIN_OWNERS) + CUS / XCDS - 1u) / (CUS / XCDS);
    const double fill = (double)u.units * 0.5 * ((double)u.n_max + (double)u.n_min) / ((double)CHAIN_OWNERS * (double)(CUS * rounds));
    const bool together = chain_together(u.units, u.n_max) > 1u;
    return rounds >= 2u && u.n_max >= (together ? 900u : 4000u) && fill >= (together && u.n_max >= 2000u ? 0.75 : 0.84);
}

// ---- 8-bit attention, any-resolution mode: do most tiles of 64 positions hold padding, on a walk of enough tiles?  Where the columns are padded every line
// of positions ends in some (lines of more than two tiles aside); where only lines are, every frame does, once in frame / 64 tiles.  The initial accumulators
// are waited for in front of a tile's first product, which short walks do not hide.  Attention alone, added where needed -> initial accumulator, us, units of
// positions, head_dim 128: 360x81 8.92 -> 9.83, 160x128 8.10 -> 8.30, 128x224 10.02 -> 10.36, 80x192 9.70 -> 9.72, 80x256 11.00 -> 10.78, 12x256 9.67 -> 9.34,
// 80x384 13.74 -> 13.01; head_dim 64: 160x128 6.45 -> 6.49, 80x192 7.45 -> 6.79, 80x320 9.37 -> 8.21.
inline bool pads_most_tiles(int head_dim, uint32_t positions, uint32_t line, uint32_t frame, bool cols_padded, bool lines_padded) {
    if (positions < (head_dim == 128 ? 256u : 192u)) return false;
    return (cols_padded && line <= 128u) || (lines_padded && frame <= 128u);
}

// ---- row moves: how many rows of `chunks` 16-byte chunks one wavefront moves.
// Batches of 4 KiB, a single round of loads: larger ones leave less in flight and lose more the longer the rows are (16 KiB: 768 B rows 91.8 us
// instead of the 87.5 of a wavefront a row, 1008 B 122 instead of 101).  Permute, switch and unpermute of 96,768 rows together, us, a wavefront
// a row -> batches: 64 B 71.5 -> 14.8, 128 B 72.8 -> 17.7, 256 B 75 -> 31, 384 B 78.7 -> 46, 512 B 79.5 -> 55, 640 B 83.7 -> 68.5,
// 768 B 87.5 -> 80.5; from 832 B on a wavefront a row is as good or better (1008 B 101 -> 105).  And only where they leave 2048
// wavefronts, two a SIMD: with fewer rows a wavefront each is as good (128 rows of 256 B: 6.9 us against 7.3).
constexpr uint32_t BATCH_CHUNKS = 256;
constexpr uint32_t BATCH_MAX_ROW = 48;
inline uint32_t row_batch(uint32_t chunks, uint32_t n_rows) {
    uint32_t batch = chunks <= BATCH_MAX_ROW ? BATCH_CHUNKS / chunks : 1u;
    batch = batch > 64u ? 64u : batch;  // lane i finds row i
    while (batch > 1u && n_rows / batch < 2048u) batch /= 2u;
    return batch;
}

// Longer rows: parts of 64 chunks a wavefront, or of up to 128 (two loads in flight) where parts of 64 would leave more than a fifth of the
// lanes idle.  Permute, switch and unpermute together, us, a wavefront a row / parts of 64 / of 128: 80,640 rows of 80 chunks 110 / 121 / 105,
// 32,256 of 144 chunks 85.4 / 84.4 / 80.9, 81,648 of 112 chunks 150 / 147 / 153, 80,640 of 192 chunks 248 / 233 / 239, of 640 chunks
// 872 / 757 / 830.
inline uint32_t row_unroll(uint32_t chunks) {
    const uint32_t lanes = (chunks + 63u) / 64u * 64u;
    return chunks > 64u && 5u * chunks < 4u * lanes ? 2u : 1u;
}
constexpr uint32_t MAX_ROW_WAVES = 1u << 25;  // a grid holds fewer than 2^32 work items; more rows than that keep a wavefront each
// chunks a wavefront moves: equal parts of whole 128-byte lines
inline uint32_t row_span(uint32_t chunks, uint32_t n_rows, uint32_t unroll) {
    uint32_t parts = (chunks + 64u * unroll - 1u) / (64u * unroll);
    while (parts > 1u && (uint64_t)n_rows * parts > MAX_ROW_WAVES) parts = (parts + 1u) / 2u;
    return ((chunks + parts - 1u) / parts + 7u) / 8u * 8u;
}

}  // namespace skiparse

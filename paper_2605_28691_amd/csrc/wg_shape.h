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
    float fixed[3];  // prologue, pipeline fill, epilogue and merge, with k = 1..max_k workgroups on a CU
    float block[3];  // per 32-row block of the walk, the same
};

// The units of a launch: how many have any row, and the rows of the largest and of the smallest one (they differ in the any-resolution
// mode only).
struct UnitSizes {
    uint64_t units;
    uint32_t n_max, n_min;
};

constexpr uint32_t GROUP_MIN_ROWS = 64;  // a group of wavefronts needs a tile of its own: units of this size or less are not split

// The shape with the smallest estimated time: rounds over the 256 CUs, each as long as `fixed` plus the blocks of the walk at the cost
// of that many workgroups per CU.  Every cost is in units of 0.1 us, fitted to launches of every shape (see the tables).  Shapes with two
// groups are left out where the first shape, the largest, fills `split_rounds` rounds: see at the forward's tables.
template <int N>
inline int pick_shape(const ShapeCost (&cost)[N], const UnitSizes& u, float split_rounds) {
    constexpr uint64_t CUS = 256;
    const float blocks = (float)((u.n_max + 31u) / 32u);
    auto workgroups = [&](int v) { return u.units * ((u.n_max + (uint32_t)cost[v].rows - 1u) / (uint32_t)cost[v].rows); };
    const bool may_split = u.n_min > GROUP_MIN_ROWS && (float)workgroups(0) < split_rounds * (float)CUS;
    int best = 0;
    float best_t = 0.f;
    for (int v = 0; v < N; v++) {
        if (cost[v].split && !may_split) continue;
        const int k = cost[v].max_k;
        const uint64_t wgs = workgroups(v), per_round = CUS * (uint64_t)k, rounds = wgs / per_round, rem = wgs % per_round;
        float t = (float)rounds * (cost[v].fixed[k - 1] + blocks * cost[v].block[k - 1]);
        if (rem != 0) {
            const uint64_t last = (rem - 1u) / CUS;
            t += cost[v].fixed[last] + blocks * cost[v].block[last];
        }
        if (v == 0 || t < best_t) {
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
};

// Costs fitted to launches of every shape over 4..1100 units of 8..80,640 tokens.  Measured, always Q256 -> picked, us at head_dim 128, units x
// tokens: 48x390 18.6 -> 13.5, 160x960 101 -> 88, 24x2600 134 -> 85, 48x2600 213 -> 165, 1x8190 166 -> 96, 1x20160 401 -> 236, 4x20160
// 948 -> 830; 192x240 (16.5), 84x512 (21.3), 48x960 (32) and 48x8190 (1400) keep it.  At head_dim 64: 24x2600 88 -> 52, 4x20160 640 -> 499,
// 160x4000 865 -> 718, 160x20160 18,550 -> 17,220; 103x377 (11.8) keeps it.
//   * Two Q128 workgroups that start together on a CU wait for the same loads, so the first round costs them more than one alone:
//     their `fixed` is larger.  With one figure for both the rule took Q128 for 192x240 (17.3), 84x512 (22.5), 225x216 (17.7 against 16.8).
//   * Two groups stream K and V at two places and move 4 % more per MFMA; what they gain is the idle part of the last round, and that
//     counts only while there are few rounds: many are spread by the power limit (the clock rises as the chip empties).  In units of Q256
//     rounds, Q256 / Q128_SPLIT, us: 1.2 948 / 830, 1.5 581 / 549, 2.5 1517 / 1509 (Q128: 1498), 6.2 3777 / 3885 (20x20160), 6.5 5738 / 6029
//     (14x30240), 6.2 7649 / 7792 (10x40320), 6.2 15,380 / 15,590 (5x80640).  From two rounds on they are left out.
constexpr ShapeCost FWD_COST_128[] = {{Q256, 256, false, 1, {40.f}, {9.0f}},
                                      {Q128, 128, false, 2, {20.f, 40.f}, {5.5f, 10.0f}},
                                      {Q64_SPLIT, 64, true, 1, {25.f}, {3.9f}},
                                      {Q128_SPLIT, 128, true, 1, {45.f}, {4.7f}}};
constexpr ShapeCost FWD_COST_64[] = {{Q256, 256, false, 1, {27.f}, {5.2f}},
                                     {Q128, 128, false, 3, {15.f, 26.f, 26.f}, {3.6f, 5.7f, 7.6f}},
                                     {Q64_SPLIT, 64, true, 2, {15.f, 15.f}, {2.4f, 3.7f}},
                                     {Q128_SPLIT, 128, true, 1, {30.f}, {2.9f}}};
constexpr float FWD_SPLIT_ROUNDS = 2.0f;
inline int pick_fwd_shape(int head_dim, const UnitSizes& u) {
    return pick_shape(head_dim == 128 ? FWD_COST_128 : FWD_COST_64, u, FWD_SPLIT_ROUNDS);
}

// ---- backward.  The dQ launch's owners are queries, the dK+dV launch's keys.
enum BwdShape : int {
    O256 = 1,       // 8 wavefronts, 1 group
    O128 = 2,       // 4 wavefronts, 1 group
    O64_SPLIT = 3,  // 4 wavefronts, 2 groups
};

// At head_dim 128 the dK+dV shapes with 4 wavefronts hold V in registers (one workgroup per CU).  Measured, always O256 -> picked, dQ and dK+dV
// together, us at head_dim 128, units x tokens: 16x200 39.8 -> 23, 12x700 78 -> 42, 48x390 62 -> 43, 160x960 347 -> 328, 24x2600 495 -> 328,
// 1x5000 411 -> 190, 1x20160 1534 -> 1150, 4x20160 3560 -> 3390; 48x960 (108), 30x8190 (3340), 12x20160 (7900) and 48x8190 (5190) keep it.
constexpr ShapeCost DQ_COST_128[] = {{O256, 256, false, 1, {50.f}, {13.0f}}, {O128, 128, false, 2, {40.f, 40.f}, {9.5f, 13.4f}}, {O64_SPLIT, 64, true, 1, {40.f}, {6.3f}}};
constexpr ShapeCost DQ_COST_64[] = {{O256, 256, false, 1, {35.f}, {8.0f}}, {O128, 128, false, 2, {28.f, 28.f}, {5.6f, 8.1f}}, {O64_SPLIT, 64, true, 2, {30.f, 30.f}, {3.4f, 6.0f}}};
constexpr ShapeCost DKV_COST_128[] = {{O256, 256, false, 1, {80.f}, {19.0f}}, {O128, 128, false, 1, {60.f}, {13.2f}}, {O64_SPLIT, 64, true, 1, {70.f}, {8.0f}}};
constexpr ShapeCost DKV_COST_64[] = {{O256, 256, false, 1, {50.f}, {10.0f}}, {O128, 128, false, 2, {40.f, 40.f}, {8.0f, 10.3f}}, {O64_SPLIT, 64, true, 1, {50.f}, {5.4f}}};

// The split shape has no limit here: none of 80 random training steps took longer than with 256 owners alone, and a long walk gains by it
// too (dK+dV of 1x80640, with dQ: 13.7 ms against 14.2).
inline int pick_bwd_shape(bool dkv, int head_dim, const UnitSizes& u) {
    const float no_limit = 3.4e38f;
    if (dkv) return pick_shape(head_dim == 128 ? DKV_COST_128 : DKV_COST_64, u, no_limit);
    return pick_shape(head_dim == 128 ? DQ_COST_128 : DQ_COST_64, u, no_limit);
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

}  // namespace skiparse

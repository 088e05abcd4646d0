// Which workgroup shape an attention launch gets.  A kernel exists in a few shapes that differ in the rows (queries, or keys in the
// dK+dV launch) a workgroup takes and in whether two groups of wavefronts share the walk over the other side; large workgroups move
// the least data per MFMA, small ones fill the chip when the problem is small.
#pragma once
#include <stdint.h>

namespace skiparse {

struct ShapeCost {
    int rows;        // rows of a workgroup
    int max_k;       // workgroups of this shape that one CU holds
    float fixed;     // prologue, pipeline fill, epilogue and merge
    float block[3];  // per 32-row block of the walk, with k = 1..max_k workgroups on a CU
};

// The shape with the smallest estimated time: rounds over the 256 CUs, each as long as `fixed` plus the blocks of the walk at the cost
// of that many workgroups per CU.  Every cost is in units of 0.1 us, fitted to launches of every shape (see the tables at the kernels).
// `n` is the number of rows of the largest unit; the shapes from `first_split` on have two groups and are left out unless `may_split`.
template <int N>
inline int pick_shape(const ShapeCost (&cost)[N], uint64_t n_units, uint32_t n, int first_split, bool may_split) {
    constexpr uint64_t CUS = 256;
    const float blocks = (float)((n + 31u) / 32u);
    int best = 0;
    float best_t = 0.f;
    for (int v = 0; v < N; v++) {
        if (v >= first_split && !may_split) continue;
        const uint64_t wgs = n_units * ((n + (uint32_t)cost[v].rows - 1u) / (uint32_t)cost[v].rows);
        const uint64_t per_round = CUS * (uint64_t)cost[v].max_k, rounds = wgs / per_round, rem = wgs % per_round;
        float t = (float)rounds * (cost[v].fixed + blocks * cost[v].block[cost[v].max_k - 1]);
        if (rem != 0) t += cost[v].fixed + blocks * cost[v].block[(rem - 1u) / CUS];
        if (v == 0 || t < best_t) {
            best = v;
            best_t = t;
        }
    }
    return best;
}

}  // namespace skiparse

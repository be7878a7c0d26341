// Score of a prompt group (Appendix B: the full method aggregates scores by
// the mean within prompt groups). Consecutive trajectories form the groups:
// group g holds trajectories [go[g], go[g+1]), offsets clamped to [0, n].
#pragma once

#include "device_util.hpp"
#include "score_math.hpp"

#pragma clang fp contract(off)

namespace pace {

// The members' scores added in member order starting from 0, then one
// division by the member count; an empty group scores 0. Members are loaded
// kGroupLoad at a time while there are that many, then eight at a time (one
// round trip each); the additions keep member order. One group of 8192 members:
// 209 us a group step, eight at a time 394.
// kJoin: score is join.ws.traj, where members summed in pieces hold a mark.
constexpr int kGroupLoad = 16;
template <bool kJoin>
__device__ __forceinline__ double group_mean(const double *__restrict__ score, int64_t n,
                                             const int64_t *__restrict__ go, int64_t g, const ScoreJoin &join) {
    const int64_t lo = clamp64(go[g], 0, n), hi = clamp64(go[g + 1], 0, n);
    double sum = 0.0;
    int64_t b = lo;
    for (; b + kGroupLoad <= hi; b += kGroupLoad) {
        double x[kGroupLoad];
#pragma unroll
        for (int k = 0; k < kGroupLoad; ++k) x[k] = score[b + k];
        if constexpr (kJoin) {
            join_marked(x, join);
        }
#pragma unroll
        for (int k = 0; k < kGroupLoad; ++k) sum = sum + x[k];
    }
    for (; b < hi; b += 8) {
        double x[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) x[k] = b + k < hi ? score[b + k] : 0.0;
        if constexpr (kJoin) {
            join_marked(x, join);
        }
#pragma unroll
        for (int k = 0; k < 8; ++k)
            if (b + k < hi) sum = sum + x[k];
    }
    return (hi > lo) ? sum / (double)(hi - lo) : 0.0;
}

}  // namespace pace

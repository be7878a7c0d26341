// The rules on sizes by which the host takes one path or another. Plain C++
// without HIP, so that the tests compile them and choose their pools by them.
#pragma once

#include <stdint.h>

namespace pace {

// Pools up to this size are selected by the multi-workgroup rank-by-counting
// kernel; larger pools by the single-workgroup radix select.
constexpr int64_t kRankMaxN = 8192;

// ---- scores by trajectory (score_traj.hip) ----------------------------------
constexpr int64_t kTrajCap = 65536;                // tokens one workgroup of four or eight waves sums, at least
constexpr int64_t kTrajOverMax = 4096;             // piece workgroups, at most (the cap grows instead)
constexpr int64_t kTrajFillWaves = 4096;           // waves that few trajectories are spread over

// Waves that take a trajectory, from the mean length: enough bytes for each
// that its start and end (about 3 us) hide under the others' streams, and
// enough waves for the chip when there are few trajectories. Whole steps, 1 / 2
// / 4 / 8 waves: 8192 trajectories of 1464 tokens 38.9 / 39.4 / 41.4 / 53.0 us,
// of 1953 42.0 / 42.2 / 43.4 / 54.5, 8000 of 3500 54.3 / 54.0 / 53.8 / 63.0,
// 4096 of 6103 42.0 / 41.0 / 39.4 / 41.4, of 12,207 75.7 / 75.0 / 70.6 / 67.1.
inline int traj_waves(int64_t n, int64_t n_tokens) {
    const int64_t mean = n_tokens / n;
    const int want = mean >= 8192 ? 8 : (mean >= 2560 ? 4 : (mean >= 1536 ? 2 : 1));
    int fill = 1;
    while (fill < 8 && fill * 2 * n <= kTrajFillWaves) fill *= 2;
    return want > fill ? want : fill;
}

// Whether the score is formed by trajectory rather than over equal chunks of
// tokens. Chunks remain for many short trajectories, where a trajectory does
// not fill a wave's loads: 16,384 trajectories of 2500 tokens take 75 us a step
// by chunks and 78 by trajectory, of 3200 90.4 and 89.2, 8200 of 5000 69 and 65.
inline bool score_by_traj(int64_t n, int64_t n_tokens) { return n <= kRankMaxN || n_tokens / n >= 3072; }

// The most tokens that one workgroup then sums.
inline int64_t score_traj_cap(int64_t n, int64_t n_tokens) {
    if (n == 0) return kTrajCap;
    const int kw = traj_waves(n, n_tokens);
    const int64_t least = kw >= 4 ? kTrajCap : kTrajCap / 4 * kw;
    const int64_t per = n_tokens / kTrajOverMax;
    return per <= least ? least : (per + least - 1) / least * least;
}

// Whether a thread's sum of tags + 1 stays below 2^32: tags are at most V (a
// precondition), and a thread sums at most cap / (64 waves) of them.
inline bool score_traj_narrow(int64_t n, int64_t n_tokens, int32_t V) {
    return (int64_t)V + 1 <= ((((int64_t)1 << 32) - 1) / (score_traj_cap(n, n_tokens) / (64 * traj_waves(n, n_tokens))));
}

// ---- scores over chunks of tokens (score.hip) -------------------------------
// Arithmetic of the reduction; tags are at most V, so tag + 1 <= V + 1.
//   kPacked  every tag + 1 < 2^15: sum and count in one 32-bit number
//   kNarrow  every tag + 1 < 2^24: 32-bit sums of a window, counts apart
//   kWideTags  64-bit sums
enum ReduceMode : int { kPacked = 0, kNarrow = 1, kWideTags = 2 };
inline ReduceMode reduce_mode(int32_t V) {
    return (int64_t)V < (1 << 15) - 1 ? kPacked : ((int64_t)V < (1 << 24) - 1 ? kNarrow : kWideTags);
}

// ---- prompt groups (group.hip) -----------------------------------------------
// Group means formed inside the rank over groups (at most kRankMaxN groups):
// every rank workgroup (one per kRankQ groups) reads all member scores, so the
// group step does that while ceil(ng / kRankQ) * n stays within kGroupRankLoads,
// and makes a separate pass of group means before the rank beyond.
constexpr int kRankQ = 16;              // targets per rank workgroup
constexpr int64_t kGroupRankLoads = (int64_t)1 << 21;
inline bool group_means_in_rank(int64_t n, int64_t ng) { return (ng + kRankQ - 1) / kRankQ * n <= kGroupRankLoads; }

// ---- small filter steps (compact.hip) ----------------------------------------
inline int64_t expected_kept(int64_t n, int64_t n_tokens, int64_t kept) {
    return n > 0 ? (int64_t)((double)n_tokens * ((double)kept / (double)n)) : 0;
}

// Whether the selection and compaction of a filter step go in one launch. Every
// workgroup repeats the ranking, so it is for batches that a few hundred
// workgroups copy: expected kept tokens times columns up to kSmallMaxCopy, twice
// that for at most half as many trajectories. Three launches / two, us a step:
// 64 trajectories, 70K tokens 16.4 / 13.4; 64, 1.5M 16.0 / 14.3; 256, 1M 16.1 /
// 14.1; 256, 2M 16.0 / 18.2; 256, 1M in three columns 17.0 / 21.3.
constexpr int64_t kSmallMaxN = 256;
constexpr int64_t kSmallMaxCopy = (int64_t)1 << 19;
inline bool small_step_ok(int64_t n, int64_t n_tokens, int n_cols, int64_t budget) {
    const int64_t most = kSmallMaxCopy * (n <= kSmallMaxN / 2 ? 2 : 1) / (n_cols > 0 ? n_cols : 1);
    return n <= kSmallMaxN && expected_kept(n, n_tokens, n - budget) <= most;
}

}  // namespace pace

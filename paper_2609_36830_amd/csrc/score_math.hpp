// Per-trajectory score of the PACE filter (Sec. 2, Sec. 3.2), as the
// finalize kernel forms it from the reduction's pieces.
//
//   T      generated (tag != -1) tokens                        Eq. (1)
//   S      sum over them of (c - tag) = c T - sum(tag), exact   Eq. (2)
//   K_wait = V - c,  K_gen = S / T (0 when T = 0)               Eq. (2)
//   F      = a^g / (a^g + (W - a)^g), a = #{w <= s_pre}         Eq. (8), (9)
//   M      = (w_wait * K_wait) + (F * K_gen)                    Eq. (6), (7)
// Every floating-point operation is one IEEE binary64 round-to-nearest step
// in this order (contraction is off for every translation unit).
#pragma once

#include "device_util.hpp"
#include "kernels.hpp"

#pragma clang fp contract(off)

namespace pace {

struct TrajScore {
    int64_t S, T;
    double score;
};

// The reduce kernel leaves, per trajectory, the sum of (tag + 1) and the
// generated-token count of the piece in the chunk holding its first token
// (part_*) and of the piece in every later chunk it covers (carry_*).
struct TrajPieces {
    uint64_t sp;   // sum of (tag + 1) over generated tokens
    int64_t T;     // generated tokens
};

// Chunk holding token position p >= 0. The chunk length is a multiple of
// kScoreChunkAlign = 2^8, so p / chunk_len = (p >> 8) / (chunk_len >> 8);
// with narrow (every position below 2^40) that is a 32-bit division.
__device__ __forceinline__ int64_t chunk_of(int64_t p, int64_t chunk_len, bool narrow) {
    static_assert(kScoreChunkAlign == 256, "chunk lengths are multiples of 2^8");
    if (narrow) return (int64_t)((uint32_t)(p >> 8) / (uint32_t)(chunk_len >> 8));
    return p / chunk_len;
}

// Pieces of trajectory i covering tokens [lo, hi): its part and the carries
// of chunks lo / chunk_len + 1 .. (hi - 1) / chunk_len. The first kCarryBatch
// carries are loaded together (one round trip); longer spans loop.
constexpr int kCarryBatch = 4;
__device__ __forceinline__ TrajPieces gather_pieces(
    int64_t i, int64_t lo, int64_t hi, const uint64_t *__restrict__ part_sum,
    const int64_t *__restrict__ part_cnt, const uint64_t *__restrict__ carry_sum,
    const int64_t *__restrict__ carry_cnt, int64_t chunk_len, bool narrow) {
    TrajPieces p{0, 0};
    if (hi > lo) {
        p.sp = part_sum[i];
        p.T = part_cnt[i];
        const int64_t first = chunk_of(lo, chunk_len, narrow) + 1;
        const int64_t last = chunk_of(hi - 1, chunk_len, narrow);
        uint64_t cs[kCarryBatch];
        int64_t cc[kCarryBatch];
#pragma unroll
        for (int u = 0; u < kCarryBatch; ++u) {
            const bool in = first + u <= last;
            cs[u] = in ? carry_sum[first + u] : 0;
            cc[u] = in ? carry_cnt[first + u] : 0;
        }
#pragma unroll
        for (int u = 0; u < kCarryBatch; ++u) {
            p.sp += cs[u];
            p.T += cc[u];
        }
        for (int64_t ch = first + kCarryBatch; ch <= last; ++ch) {
            p.sp += carry_sum[ch];
            p.T += carry_cnt[ch];
        }
    }
    return p;
}

// Prefix weight F from a = #{w in window : w <= s_pre}.
__device__ __forceinline__ double prefix_weight(int64_t a, int64_t W, int gamma) {
    int64_t A = 1, B = 1;
    for (int g = 0; g < gamma; ++g) {
        A *= a;
        B *= (W - a);
    }
    return (double)A / (double)(A + B);
}

// Score of one trajectory from its sums and prefix weight.
__device__ __forceinline__ TrajScore score_from_weight(TrajPieces pc, int64_t c, int32_t V, double F, double w_wait) {
    const uint64_t sp = pc.sp;
    const int64_t T = pc.T;
    // sp = sum(tag) + T over generated tokens
    const int64_t sum_tag = (int64_t)(sp - (uint64_t)T);
    TrajScore r;
    r.T = T;
    r.S = c * T - sum_tag;
    const double k_wait = (double)((int64_t)V - c);
    const double k_gen = (T > 0) ? (double)r.S / (double)T : 0.0;
    const double wait_term = w_wait * k_wait;
    const double gen_term = F * k_gen;
    r.score = wait_term + gen_term;
    return r;
}

// Count of the ascending window's entries <= s_pre.
__device__ __forceinline__ int64_t window_count(const double *win, int64_t W, double s_pre) {
    int64_t a_lo = 0, a_hi = W;
    while (a_lo < a_hi) {
        const int64_t mid = (a_lo + a_hi) >> 1;
        if (win[mid] <= s_pre) a_lo = mid + 1; else a_hi = mid;
    }
    return a_lo;
}

// Score of one trajectory from its pieces.
__device__ __forceinline__ TrajScore score_from_pieces(
    TrajPieces pc, int64_t c, int32_t V, bool use_prefix, double s_pre, const double *win, int64_t W,
    double w_wait, int gamma) {
    const bool with_f = use_prefix && !__builtin_isnan(s_pre);
    return score_from_weight(pc, c, V, with_f ? prefix_weight(window_count(win, W, s_pre), W, gamma) : 1.0, w_wait);
}

// ---- scores formed by trajectory (score_traj.hip) ----------------------------
// A trajectory of more than cap tokens, starting in tokens [k cap, (k + 1) cap),
// is summed in np pieces of cap tokens. Its entry of ws.traj is join_mark(k, np)
// (a NaN, which no score is), and carry slots hold: 4 k its first piece's sums,
// 4 (k + p) + 1 those of piece p >= 1, 4 k + 2 the prefix weight F and the
// completion version. (Two such trajectories cannot start within cap tokens, so
// no slot is used twice.) A reader that meets the mark needs one round trip:
// with the slots found through the offsets and F through a search of the window
// it took five, and 24 such trajectories among 3750 cost the rank 8 us.
constexpr int kJoinSlots = 4;
constexpr uint64_t kJoinMark = 0x7ffc000000000000ull;
__device__ __forceinline__ double join_mark(int64_t k, int64_t np) {
    return __longlong_as_double((long long)(kJoinMark | ((uint64_t)k << 24) | (uint64_t)np));
}
__device__ __forceinline__ bool is_join_mark(double s) {
    return ((uint64_t)__double_as_longlong(s) >> 48) == (kJoinMark >> 48);
}

__device__ inline TrajScore joined_score(double mark, const ScoreJoin &j) {
    const uint64_t m = (uint64_t)__double_as_longlong(mark);
    const int64_t k = (int64_t)((m >> 24) & 0xffffff), np = (int64_t)(m & 0xffffff);
    const uint64_t *__restrict__ cs = j.ws.carry_sum;
    const int64_t *__restrict__ cc = j.ws.carry_cnt;
    const double F = __longlong_as_double((long long)cs[kJoinSlots * k + 2]);
    const int64_t c = cc[kJoinSlots * k + 2];
    TrajPieces p{cs[kJoinSlots * k], cc[kJoinSlots * k]};
    for (int64_t b = 1; b < np; b += kCarryBatch) {
        uint64_t xs[kCarryBatch];
        int64_t xc[kCarryBatch];
#pragma unroll
        for (int u = 0; u < kCarryBatch; ++u) {
            const bool in = b + u < np;
            xs[u] = in ? cs[kJoinSlots * (k + b + u) + 1] : 0;
            xc[u] = in ? cc[kJoinSlots * (k + b + u) + 1] : 0;
        }
#pragma unroll
        for (int u = 0; u < kCarryBatch; ++u) {
            p.sp += xs[u];
            p.T += xc[u];
        }
    }
    return score_from_weight(p, c, j.a.V, F, j.a.w_wait);
}

// Replaces the marks among x by their scores: every lane its first one at a
// time, so that a wave takes as many round trips as one lane has marks.
template <int N>
__device__ __forceinline__ void join_marked(double (&x)[N], const ScoreJoin &j) {
    // Most often there are none: the least distance above the marks tells, at a
    // third of the search's instructions (one group of 8192 members 467 -> 394 us).
    uint32_t d = ~0u;
#pragma unroll
    for (int k = 0; k < N; ++k) {
        const uint32_t e = (uint32_t)((uint64_t)__double_as_longlong(x[k]) >> 32) - (uint32_t)(kJoinMark >> 32);
        d = e < d ? e : d;
    }
    if (d >> 16) return;
    while (true) {
        int at = -1;
        double m = 0.0;
#pragma unroll
        for (int k = N - 1; k >= 0; --k) {
            if (is_join_mark(x[k])) {
                at = k;
                m = x[k];
            }
        }
        if (at < 0) return;
        const double y = joined_score(m, j).score;
#pragma unroll
        for (int k = 0; k < N; ++k) x[k] = k == at ? y : x[k];
    }
}

// joined_score of trajectory i, written to its outputs.
__device__ inline double write_joined(int64_t i, double mark, const ScoreJoin &j) {
    const TrajScore r = joined_score(mark, j);
    j.a.score[i] = r.score;
    if (j.a.gen_sum) j.a.gen_sum[i] = r.S;
    if (j.a.gen_count) j.a.gen_count[i] = r.T;
    return r.score;
}

// The smallest and largest key of a workgroup of kFinGroup trajectories (in:
// the thread holds one), the range the wide selection histograms; workgroup 0
// clears that selection's level-0 histogram (hist0).
__device__ __forceinline__ void key_extremes(uint64_t key, bool in, uint64_t *__restrict__ mmin,
                                             uint64_t *__restrict__ mmax, uint32_t *__restrict__ hist0) {
    if (blockIdx.x == 0)
        for (int b = threadIdx.x; b < (1 << kCutBits); b += kFinGroup) hist0[b] = 0u;
    __shared__ uint64_t wl[kFinGroup / kWave], wh[kFinGroup / kWave];
    const uint64_t lo = wave_min_u64(in ? key : ~0ull), hi = wave_max_u64(in ? key : 0ull);
    if (lane_id() == 0) {
        wl[threadIdx.x / kWave] = lo;
        wh[threadIdx.x / kWave] = hi;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        uint64_t a = ~0ull, b = 0;
        for (int w = 0; w < kFinGroup / kWave; ++w) {
            a = wl[w] < a ? wl[w] : a;
            b = wh[w] > b ? wh[w] : b;
        }
        mmin[blockIdx.x] = a;
        mmax[blockIdx.x] = b;
    }
}

}  // namespace pace

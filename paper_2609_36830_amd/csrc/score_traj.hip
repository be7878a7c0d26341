// pace_score by trajectory for gfx950: one workgroup reads a whole
// trajectory's tags, sums them and forms its score (Sec. 2 and 3.2, Eq. (1),
// (2), (6)-(9)), so that no per-chunk pieces go through memory and no second
// kernel waits for them.
//
// HBM-bound, 4 bytes per token. Every thread keeps eight 16-byte loads in
// flight (each dword-aligned, so a trajectory may start anywhere); a partial
// batch reads clamped addresses and masks, so no load sits behind a branch.
// The workgroups of the other trajectories hide one's start (its offsets) and
// end (the sums over the waves, the window count, two divisions), and the
// order in which the chip finishes them evens out their lengths. The window
// entries at or below the prefix score are found by the first wave beside the
// tags' loads (WindowSearch).
//
// A trajectory of more than `cap` tokens would leave one workgroup at work
// alone: its first cap tokens are its workgroup's, and workgroup n + k takes
// the piece that starts in tokens [k cap, (k + 1) cap), if any: only the
// trajectory holding token k cap can have one there. Their sums are joined by
// the kernel that reads the scores next (the rank) or by score_join.
//
// Against equal token chunks per wave with the pieces added up by a second
// kernel, calls back to back: 64 trajectories, 70K tokens 11.0 -> 3.8 us; 1024,
// 3.8M 11.1 -> 6.6; 2048, 20M 19.0 -> 15.7; 4096, 50.1M 39.9 -> 35.0 us (5.7
// TB/s).
#include "device_util.hpp"
#include "kernels.hpp"
#include "score_math.hpp"

#pragma clang fp contract(off)

namespace pace {

namespace {

constexpr int kTU = 8;                             // 16-byte loads in flight per thread

// Sums of one thread: the tags + 1 and the generated tokens.
struct Narrow {                                    // a thread's tags, each at most V + 1, sum below 2^32
    uint32_t s = 0, c = 0;
    __device__ __forceinline__ void add(uint32_t x0, uint32_t x1, uint32_t x2, uint32_t x3) {
        s += x0 + x1 + x2 + x3 + 4u;               // a masked tag (-1) adds 0
        c += 4u - ((x0 >> 31) + (x1 >> 31) + (x2 >> 31) + (x3 >> 31));
    }
};
struct Wide {
    uint64_t s = 0;
    uint32_t c = 0;
    __device__ __forceinline__ void add(uint32_t x0, uint32_t x1, uint32_t x2, uint32_t x3) {
        const uint32_t u0 = x0 + 1u, u1 = x1 + 1u, u2 = x2 + 1u, u3 = x3 + 1u;
        s += (uint64_t)u0 + u1 + u2 + u3;
        c += (u0 != 0u) + (u1 != 0u) + (u2 != 0u) + (u3 != 0u);
    }
};

// U vectors of four tags from p on, `stride` tokens apart, of a piece ending
// at e (at least four tokens long). kLast: vectors may reach past e; they are
// read from e - 4 and the tokens before p masked.
template <int U, bool kLast, typename A>
__device__ __forceinline__ void add_tags(const int32_t *__restrict__ tags, int64_t p, int64_t e, int stride, A &acc) {
    uint4 x[U];
    int d[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        int64_t q = p + (int64_t)u * stride;
        if (kLast) {
            const int64_t over = q - (e - 4);
            d[u] = over <= 0 ? 0 : (over < 4 ? (int)over : 4);
            q = over <= 0 ? q : e - 4;
        }
        x[u] = load_a4(tags + q);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        if (kLast) {
            x[u].x = d[u] > 0 ? ~0u : x[u].x;
            x[u].y = d[u] > 1 ? ~0u : x[u].y;
            x[u].z = d[u] > 2 ? ~0u : x[u].z;
            x[u].w = d[u] > 3 ? ~0u : x[u].w;
        }
        acc.add(x[u].x, x[u].y, x[u].z, x[u].w);
    }
}

// Count of the ascending window's entries <= s, by a 64-way search of one wave
// (the lanes' probes of a level are one load). No level costs a round trip of
// its own for windows of up to 4096 entries: the top level's entries are loaded
// with the offsets, before s is known, and the last level's before the tags,
// which come after them. Counting all entries beside the tags, one per thread,
// loaded the whole window in every workgroup: a step of 8192 trajectories of 500
// tokens took 30.8 us with 512 entries and 45.6 with 4096, now 29.4 with either.
struct WindowSearch {
    int64_t at = 0, len = 0;    // the count lies in [at, at + len]
    double x = 0.0;             // the lane's entry of the level at hand
    __device__ __forceinline__ static int64_t stride(int64_t len) { return (len + kWave - 1) / kWave; }
    __device__ __forceinline__ void load(const double *__restrict__ w, int64_t st) {
        const int64_t k = (int64_t)lane_id() * st;
        if (k < len) x = w[at + k];
    }
    __device__ __forceinline__ void top(const double *__restrict__ w, int64_t W) {
        len = W;
        load(w, stride(len));
    }
    __device__ __forceinline__ void down(const double *__restrict__ w, double s) {
        while (len > kWave) {
            const int64_t st = stride(len);
            const int64_t le = __popcll(ballot((int64_t)lane_id() * st < len && x <= s));
            if (le == 0) {
                len = 0;
                return;
            }
            at += (le - 1) * st;
            len = len - (le - 1) * st < st ? len - (le - 1) * st : st;
            load(w, stride(len));
        }
    }
    __device__ __forceinline__ int64_t count(double s) const {
        return at + __popcll(ballot(lane_id() < len && x <= s));
    }
};

template <typename A, int kW>
__global__ __launch_bounds__(kW * kWave) void score_traj_kernel(const int32_t *__restrict__ tags, ScoreArgs a,
                                                               ScoreWorkspace ws, int64_t cap) {
    constexpr int kT = kW * kWave;
    constexpr int kStride = kT * 4;
    __shared__ uint64_t w_s[kW];
    __shared__ uint32_t w_c[kW];
    const int t = threadIdx.x, lane = lane_id();
    WindowSearch win;
    if (a.use_prefix && t < kWave) win.top(a.window, a.W);
    // The trajectory, and its tokens [p, e) that are this workgroup's.
    int64_t i = blockIdx.x, p, e, slot = -1, n_pieces = 1;
    bool whole = true;
    if (i < a.n) {
        const int64_t lo = readlane_i64(clamp64(a.off[i], 0, a.NT), 0);
        const int64_t hi = readlane_i64(clamp64(a.off[i + 1], 0, a.NT), 0);
        p = lo;
        e = hi;
        if (hi - lo > cap) {
            e = lo + cap;
            whole = false;
            slot = kJoinSlots * (lo / cap);
            n_pieces = (hi - lo + cap - 1) / cap;
        }
    } else {
        // One wave searches: most windows hold no piece, and eight waves'
        // searches of each cost the 50M-token step 0.2 us.
        __shared__ int64_t found[3];
        const int64_t k = i - a.n;
        if (t < kWave) {
            int64_t at = wave_last_le(a.off, a.n, k * cap), p0 = 0, e0 = 0;
            if (at >= 0 && at < a.n) {
                const int64_t lo = clamp64(a.off[at], 0, a.NT), hi = clamp64(a.off[at + 1], 0, a.NT);
                if (k * cap > lo) {
                    p0 = lo + (k * cap - lo + cap - 1) / cap * cap;
                    e0 = p0 + cap < hi ? p0 + cap : hi;
                }
            }
            if (t == 0) {
                found[0] = at;
                found[1] = p0;
                found[2] = e0;
            }
        }
        __syncthreads();
        i = readlane_i64(found[0], 0);
        p = readlane_i64(found[1], 0);
        e = readlane_i64(found[2], 0);
        if (p >= e) return;
        whole = false;
        slot = kJoinSlots * k + 1;
    }
    // Loads that the end of the kernel needs go first.
    const bool first = whole || (slot % kJoinSlots) == 0;      // holds the trajectory's start
    const double s_pre = first && a.use_prefix ? a.prefix[i] : __builtin_nan("");
    const int64_t c = a.completion[i];
    const bool with_f = !__builtin_isnan(s_pre);
    if (with_f && t < kWave) win.down(a.window, s_pre);

    A acc;
    if (e - p >= 4) {
        for (; p + kTU * kStride <= e; p += kTU * kStride) add_tags<kTU, false>(tags, p + t * 4, e, kStride, acc);
        if (p + 6 * kStride < e) add_tags<8, true>(tags, p + t * 4, e, kStride, acc);
        else if (p + 4 * kStride < e) add_tags<6, true>(tags, p + t * 4, e, kStride, acc);
        else if (p + 2 * kStride < e) add_tags<4, true>(tags, p + t * 4, e, kStride, acc);
        else if (p < e) add_tags<2, true>(tags, p + t * 4, e, kStride, acc);
    } else if (t < e - p) {
        acc.add((uint32_t)tags[p + t], ~0u, ~0u, ~0u);
    }
    const uint64_t s = wave_sum_u64((uint64_t)acc.s);
    const uint32_t cn = (uint32_t)readlane_i32((int32_t)wave_incl_scan_u32(acc.c), kWave - 1);
    const int64_t at_most = with_f && t < kWave ? win.count(s_pre) : 0;
    if (lane == 0) {
        w_s[t / kWave] = s;
        w_c[t / kWave] = cn;
    }
    __syncthreads();
    if (t != 0) return;
    TrajPieces pc{0, 0};
#pragma unroll
    for (int w = 0; w < kW; ++w) {
        pc.sp += w_s[w];
        pc.T += (int64_t)w_c[w];
    }
    double F = 1.0;
    if (with_f) F = prefix_weight(at_most, a.W, a.gamma);
    if (!whole) {
        ws.carry_sum[slot] = pc.sp;
        ws.carry_cnt[slot] = pc.T;
        if (first) {
            ws.carry_sum[slot + 2] = (uint64_t)__double_as_longlong(F);
            ws.carry_cnt[slot + 2] = c;
            ws.traj[i] = join_mark(slot / kJoinSlots, n_pieces);
        }
        return;
    }
    const TrajScore r = score_from_weight(pc, c, a.V, F, a.w_wait);
    ws.traj[i] = r.score;
    a.score[i] = r.score;
    if (a.gen_sum) a.gen_sum[i] = r.S;
    if (a.gen_count) a.gen_count[i] = r.T;
}

// The carries, one per kScoreChunkMin tokens, hold kJoinSlots per window of
// cap >= kTrajCap / 4 tokens, the last window's included, once there are more
// than cap tokens; window and piece numbers fit the mark's 24 bits.
static_assert(kTrajCap / 4 / kScoreChunkMin >= 2 * kJoinSlots, "carry slots");
static_assert(kTrajOverMax * 4 < (1 << 24), "window numbers in the mark");

// Trajectories of more than cap tokens; kMinMax as in score_finalize.
template <bool kMinMax>
__global__ __launch_bounds__(kFinGroup) void score_join_kernel(ScoreJoin j, uint64_t *__restrict__ mmin,
                                                              uint64_t *__restrict__ mmax,
                                                              uint32_t *__restrict__ hist0) {
    const int64_t i = (int64_t)blockIdx.x * kFinGroup + threadIdx.x;
    const bool in = i < j.a.n;
    double s = in ? j.ws.traj[i] : 0.0;
    if (in && is_join_mark(s)) s = write_joined(i, s, j);
    if constexpr (kMinMax) key_extremes(score_key(s), in, mmin, mmax, hist0);
}

}  // namespace

hipError_t launch_score_traj(const int32_t *tags, const ScoreArgs &a, const ScoreWorkspace &ws, hipStream_t stream) {
    if (a.n == 0) return hipSuccess;
    const int kw = traj_waves(a.n, a.NT);
    const int64_t cap = score_traj_cap(a.n, a.NT);
    const int64_t over = a.NT > cap ? (a.NT + cap - 1) / cap : 0;
    const dim3 grid((unsigned)(a.n + over));
    static_assert(kWave == 64, "score_traj_narrow");
    const bool narrow = score_traj_narrow(a.n, a.NT, a.V);
#define PACE_TRAJ(W)                                                                                              \
    do {                                                                                                          \
        if (narrow) return launch(kPhaseReduce, score_traj_kernel<Narrow, W>, grid, dim3((W) * kWave), stream, tags, \
                                  a, ws, cap);                                                                    \
        return launch(kPhaseReduce, score_traj_kernel<Wide, W>, grid, dim3((W) * kWave), stream, tags, a, ws, cap); \
    } while (0)
    if (kw == 8) PACE_TRAJ(8);
    if (kw == 4) PACE_TRAJ(4);
    if (kw == 2) PACE_TRAJ(2);
    PACE_TRAJ(1);
#undef PACE_TRAJ
}

hipError_t launch_score_join(const ScoreArgs &a, const ScoreWorkspace &ws, hipStream_t stream, uint64_t *mmin,
                             uint64_t *mmax, uint32_t *hist0) {
    const int64_t cap = score_traj_cap(a.n, a.NT);
    if (a.n == 0 || (!mmin && a.NT <= cap)) return hipSuccess;
    const dim3 grid((unsigned)((a.n + kFinGroup - 1) / kFinGroup));
    if (mmin)
        return launch(kPhaseFinalize, score_join_kernel<true>, grid, dim3(kFinGroup), stream, ScoreJoin{a, ws, cap},
                      mmin, mmax, hist0);
    return launch(kPhaseFinalize, score_join_kernel<false>, grid, dim3(kFinGroup), stream, ScoreJoin{a, ws, cap}, mmin,
                  mmax, hist0);
}

}  // namespace pace

// pace_validate kernels for gfx950: device check of the preconditions of
// Lemma 1 (every generated token has v_t <= c(tau) <= j; versions are
// non-negative) and of the CSR layout and prefix window. One kernel clears the
// error word; the other's first workgroups check offsets, completion versions
// and the window, one entry per thread, and the rest check the tags, one wave
// per chunk of tokens.
#include "../../include/pace.h"
#include "device_util.hpp"
#include "kernels.hpp"

namespace pace {

namespace {

constexpr int64_t kValChunk = 8192;   // tokens per wave
constexpr int64_t kLaneMean = 128;    // trajectories of at most this many tokens on average: one per lane
constexpr int64_t kLaneStep = 16;     // tokens per lane and round trip

__global__ void validate_init_kernel(int32_t *err) { *err = 0; }

// Offsets and completion versions of trajectory i, and window entry i.
__device__ __forceinline__ int32_t meta_bits(int64_t i, const int64_t *__restrict__ off, int64_t n, int64_t NT,
                                             const int32_t *__restrict__ completion, int32_t V,
                                             const double *__restrict__ window, int64_t W) {
    int32_t bad = 0;
    if (i == 0 && (off[0] != 0 || off[n] != NT)) bad |= PACE_BAD_OFFSETS;
    if (i < n) {
        if (off[i + 1] < off[i]) bad |= PACE_BAD_OFFSETS;
        const int32_t c = completion[i];
        if (c < 0 || c > V) bad |= PACE_BAD_COMPLETION;
    }
    if (i < W) {
        const double a = window[i];
        if (__builtin_isnan(a) || (i + 1 < W && !(a <= window[i + 1]))) bad |= PACE_BAD_WINDOW;
    }
    return bad;
}

// Largest tag + 1, as an unsigned number, of tokens [a, e): below -1 it is
// huge, -1 gives 0. U vectors of four tags per lane in flight; a lane past the
// end reads the last four tags again, so no load sits behind a branch.
template <int U>
__device__ __forceinline__ uint32_t max_tag1(const int32_t *__restrict__ tags, int64_t a, int64_t e, uint32_t m) {
    const int64_t last = e - 4;
    uint4 x[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int64_t p = a + ((int64_t)u * kWave + lane_id()) * 4;
        x[u] = load_a4(tags + (p < last ? p : last));
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
        m = max(max(m, max(x[u].x + 1u, x[u].y + 1u)), max(x[u].z + 1u, x[u].w + 1u));
    return m;
}

// The tags of up to 64 short trajectories, one per active lane (ends h in
// order, from lo on, limits lim), four vectors per lane in flight. False, with
// nothing done, when they are not short or the ends are not in order; else lo
// moves to the last end. Taken one after the other each trajectory costs the
// wave a round trip, one per lane a batch costs one per kLaneStep tokens of its
// longest but reads whole lines for its vectors; so one per lane where that is
// no more round trips and kLaneMean holds. One after the other / one per lane:
// 400,000 trajectories of 5 tokens 721 / 36 us, 65,536 of 64 80 / 11, of 120 48
// / 16, of 200 36 / 44 (that is why kLaneMean); 262,144 log-normal lengths of
// 100 on average 84 / 85. A lane with no more tokens reads the vector that all
// such lanes read: reading on along its own, those 262,144 took 201 us. (Loads
// behind a branch instead, or a loop that lanes leave one by one, slow the other
// walk of the kernel down: 100,000 of 200 tokens 36 -> 42 us.)
__device__ __forceinline__ bool lane_segments(const int32_t *__restrict__ tags, int64_t NT, bool active, int64_t h,
                                              uint32_t lim, int64_t ce, int64_t &lo, int64_t front, bool &bad) {
    const uint64_t act = ballot(active);
    const int first = __ffsll((long long)act) - 1, last = 63 - __clzll((long long)act);
    const int64_t end = readlane_i64(h, last), tokens = (end < ce ? end : ce) - lo;
    if (front > lo || NT < 4 || tokens > kLaneMean * __popcll(act)) return false;
    const int up = (lane_id() - 1) << 2;
    const int64_t below = (int64_t)(((uint64_t)(uint32_t)__builtin_amdgcn_ds_bpermute(up, (int)((uint64_t)h >> 32)) << 32) |
                                    (uint32_t)__builtin_amdgcn_ds_bpermute(up, (int)(uint32_t)h));
    const int64_t a = lane_id() == first ? lo : below, e = h < ce ? h : ce;
    const int64_t len = active && e > a ? e - a : 0;
    const int64_t some = __popcll(ballot(len > 0));
    if (tokens > kLaneMean * some || ballot(active && (h < a || len > kLaneStep * some))) return false;
    for (int64_t p = a; ballot(p - a < len); p += kLaneStep) {
        uint4 x[4];
        int64_t q[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            // In the array; tokens outside [a, e) are dropped. Where a lane has
            // no more, it reads the vector that all such lanes read.
            q[u] = p + 4 * u - a < len ? p + 4 * u : lo;
            q[u] = q[u] < NT - 4 ? q[u] : NT - 4;
            x[u] = load_a4(tags + q[u]);
        }
        uint32_t m = 0;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int64_t d = q[u] - a;
            m = max(m, d >= 0 && d < len ? x[u].x + 1u : 0u);
            m = max(m, d + 1 >= 0 && d + 1 < len ? x[u].y + 1u : 0u);
            m = max(m, d + 2 >= 0 && d + 2 < len ? x[u].z + 1u : 0u);
            m = max(m, d + 3 >= 0 && d + 3 < len ? x[u].w + 1u : 0u);
        }
        bad |= m > lim;
    }
    lo = end;
    return true;
}

// Workgroups [0, n_meta): 256 entries each of the offsets, completion versions
// and window. The others: one wave per chunk of kValChunk tokens, every tag -1
// or within [0, c] of its trajectory. The wave takes the trajectories of its
// chunk in turn, 64 offsets and versions at a time in its lanes, short ones one
// per lane (lane_segments) and others one after the other, as whole vectors
// against one limit, so that it is bound by the tags' bytes: 21.7M tags in 2048 trajectories 111 us (64 tags a round
// trip, each window's offsets loaded again) -> 16.4 us.
// With malformed offsets the tag bit is that of this walk: trajectories in
// order from the one holding the chunk's first token, each from where the one
// before it ended (but not behind the 64-token window that the walk has
// reached) to its own end.
__global__ __launch_bounds__(256) void validate_kernel(
    const int32_t *__restrict__ tags, const int64_t *__restrict__ off, int64_t n, int64_t NT,
    const int32_t *__restrict__ completion, int32_t V, const double *__restrict__ window, int64_t W, int64_t n_meta,
    int64_t n_chunks, int32_t *err) {
    if ((int64_t)blockIdx.x < n_meta) {
        const int32_t bits = meta_bits((int64_t)blockIdx.x * blockDim.x + threadIdx.x, off, n, NT, completion, V, window, W);
        if (bits) atomicOr(err, bits);
        return;
    }
    const int lane = lane_id();
    const int64_t chunk = ((int64_t)blockIdx.x - n_meta) * 4 + __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    if (chunk >= n_chunks) return;
    const int64_t cs = chunk * kValChunk;
    const int64_t ce = (cs + kValChunk < NT) ? cs + kValChunk : NT;
    int64_t cur = wave_last_le(off, n, cs);
    if (cur < 0) cur = 0;             // malformed offsets are reported by the meta workgroups
    bool bad = false, started = false;
    int64_t lo = cs, front = cs;      // the walk's position, and its 64-token window
    for (; cur < n; cur += kWave) {
        const int64_t i = cur + lane;
        const int64_t h = i < n ? clamp64(off[i + 1], 0, NT) : 0;
        const int32_t cl = i < n ? completion[i] : 0;
        const uint32_t lim = cl < -1 ? 0u : (uint32_t)cl + 1u;
        const int cnt = (int)(n - cur < kWave ? n - cur : kWave);
        int k = 0;
        if (!started) {               // skip what ends at or before the chunk's start
            const uint64_t m = ballot(i < n && h > cs);
            if (!m) continue;
            k = __ffsll((long long)m) - 1;
            started = true;
        }
        if (lane_segments(tags, NT, lane >= k && lane < cnt, h, lim, ce, lo, front, bad)) {
            if (lo >= ce) break;      // the chunk is done
            front = cs + (lo - cs) / 64 * 64;
            continue;
        }
        for (; k < cnt; ++k) {
            const int64_t hi = readlane_i64(h, k);
            int64_t a = lo > front ? lo : front;
            const int64_t e = hi < ce ? hi : ce;
            if (a < e) {
                const uint32_t top = (uint32_t)readlane_i32((int32_t)lim, k);
                uint32_t m = 0;
                if (e - a < 4) {
                    if (a + lane < e) m = (uint32_t)tags[a + lane] + 1u;
                } else {
                    for (; e - a > 4 * 4 * kWave; a += 8 * 4 * kWave) m = max_tag1<8>(tags, a, e, m);
                    if (a < e) m = max_tag1<4>(tags, a, e, m);
                }
                bad |= m > top;
            }
            if (hi >= ce) {
                cur = n;              // the chunk is done
                break;
            }
            if (hi > front) front = cs + (hi - cs) / 64 * 64;
            lo = hi;
        }
    }
    if (ballot(bad) && lane == 0) atomicOr(err, PACE_BAD_TAG);
}

}  // namespace

hipError_t launch_validate(const int32_t *tags, const int64_t *offsets, int64_t n, int64_t n_tokens,
                           const int32_t *completion, int32_t V, const double *window, int64_t W,
                           int32_t *err_word, hipStream_t stream) {
    validate_init_kernel<<<1, 1, 0, stream>>>(err_word);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int64_t m = (n + 1 > W) ? n + 1 : W;
    const int64_t n_meta = (m + 255) / 256;
    const int64_t ch = n > 0 ? (n_tokens + kValChunk - 1) / kValChunk : 0;
    return launch(-1, validate_kernel, dim3((unsigned)(n_meta + (ch + 3) / 4)), dim3(256), stream, tags, offsets, n,
                  n_tokens, completion, V, window, W, n_meta, ch, err_word);
}

}  // namespace pace

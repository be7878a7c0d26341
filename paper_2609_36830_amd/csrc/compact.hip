// pace_compact kernels for gfx950: pack the kept trajectories' token spans
// into the training batch (Algorithm 1), survivors in pool order.
//
// Copy routine of the scan path: a wave copies a contiguous range of output
// elements. Output goes out as aligned 16-byte non-temporal vectors (64 lanes
// x 16 B = 1 KiB per wave window, four windows in flight); sources are read
// with plain loads, since the kept spans are often still in the last-level
// cache from the scoring pass. Inside one kept span the source is the
// destination shifted by a constant, so the source
// misalignment is wave-uniform: each lane loads the aligned 16 bytes under
// its window, takes the next 16 bytes from the neighbouring lane (lane 63
// loads them), and a byte funnel shift assembles the output vector. Windows
// that straddle span ends, the ragged tail and unaligned columns copy element
// by element.
//
// Range path (n <= kPieceMaxN): consecutive trajectories form blocks of
// kPieceBlock; per block the rank kernel (or compact_partials_kernel) has
// written the kept count and kept tokens. The packed output is cut into equal
// ranges, one workgroup per range and column (compact_range_kernel below).
//
// Wide path (8192 < n <= kWideMaxN): blocks of kWideBlock trajectories with
// two-level partials, and the packed output split evenly over one resident
// round of workgroups by merge path (compact_wide_kernel below).
//
// Scan path (larger pools): one workgroup scans the flags into the packed
// offsets, kept ids, span sources and a map from each output chunk of
// kCopyChunk elements to its first span; a second kernel copies.
#include <algorithm>

#include "device_util.hpp"
#include "kernels.hpp"
#include "score_math.hpp"

namespace pace {

namespace {

constexpr int kT = 1024;
constexpr int kNW = kT / kWave;

// ---------------------------------------------------------------------------
// Spans: packed offsets o(j) and source starts s(j) of kept span j
// ---------------------------------------------------------------------------
// Global arrays, lane k caching entry base + k.
struct GlobalSpans {
    const int64_t *oo;
    const int64_t *ss;
    int64_t n_kept;
    int64_t base, o, s;
    __device__ __forceinline__ void load(int64_t b) {
        base = b;
        const int64_t idx = b + lane_id();
        o = (idx <= n_kept) ? oo[idx] : INT64_MAX;
        s = (idx < n_kept) ? ss[idx] : 0;
    }
    __device__ __forceinline__ void ensure(int64_t j) {   // entries j and j + 1
        if (j < base || j + 1 - base >= kWave) load(j);
    }
    __device__ __forceinline__ int64_t O(int64_t j) const { return readlane_i64(o, (int)(j - base)); }
    __device__ __forceinline__ int64_t S(int64_t j) const { return readlane_i64(s, (int)(j - base)); }
};

template <int E> struct Elem;
template <> struct Elem<1> { using T = uint8_t; };
template <> struct Elem<2> { using T = uint16_t; };
template <> struct Elem<4> { using T = uint32_t; };
template <> struct Elem<8> { using T = uint64_t; };

// Bytes [shift, shift + 16) of the 32-byte little-endian string a|b
// (shift is wave-uniform).
__device__ __forceinline__ uint4 funnel16(const uint4 &a, const uint4 &b, int shift) {
    const uint32_t r = (uint32_t)(shift & 3);
#define AB(hi, lo) __builtin_amdgcn_alignbyte((hi), (lo), r)
    uint4 o;
    switch (shift >> 2) {
        case 0: o = make_uint4(AB(a.y, a.x), AB(a.z, a.y), AB(a.w, a.z), AB(b.x, a.w)); break;
        case 1: o = make_uint4(AB(a.z, a.y), AB(a.w, a.z), AB(b.x, a.w), AB(b.y, b.x)); break;
        case 2: o = make_uint4(AB(a.w, a.z), AB(b.x, a.w), AB(b.y, b.x), AB(b.z, b.y)); break;
        default: o = make_uint4(AB(b.x, a.w), AB(b.y, b.x), AB(b.z, b.y), AB(b.w, b.z)); break;
    }
#undef AB
    return o;
}

__device__ __forceinline__ uint4 shfl_down1(const uint4 &a) {
    uint4 b;
    b.x = (uint32_t)__shfl_down((int)a.x, 1, kWave);
    b.y = (uint32_t)__shfl_down((int)a.y, 1, kWave);
    b.z = (uint32_t)__shfl_down((int)a.z, 1, kWave);
    b.w = (uint32_t)__shfl_down((int)a.w, 1, kWave);
    return b;
}

// Copies packed elements [cs, ce) of one column; j is a kept span with
// o(j) <= cs (the last such, for well-formed input). Every access is checked
// against n_tokens, so malformed offsets stay in bounds.
template <int E, typename Spans>
__device__ void copy_range(const char *__restrict__ in, char *__restrict__ out, bool vec, Spans &sp,
                           int64_t n_kept, int64_t NT, int64_t cs, int64_t ce, int64_t j) {
    using T = typename Elem<E>::T;
    constexpr int VE = 16 / E;          // elements per lane vector
    constexpr int WE = kWave * VE;      // elements per wave window (1 KiB)
    constexpr int U = 4;                // windows per unrolled step
    const int lane = lane_id();
    const int64_t nbytes = NT * E;
    for (int64_t w = cs; w < ce; w += WE) {
        sp.ensure(j);
        while (j + 1 < n_kept && sp.O(j + 1) <= w) {
            ++j;
            sp.ensure(j);
        }
        const int64_t we = (w + WE < ce) ? w + WE : ce;
        const int64_t o_lo = sp.O(j), o_hi = sp.O(j + 1);
        const int64_t delta = sp.S(j) - o_lo;          // src element = dst element + delta
        const int shift = (int)((((delta * E) % 16) + 16) % 16);
        // lane 63's extra aligned vector after its own, for the last window
        auto tail_ok = [&](int64_t nwin) {
            const int64_t ab63 = (w + (nwin - 1) * WE + (int64_t)(kWave - 1) * VE + delta) * E - shift;
            return shift == 0 || ab63 + 32 <= nbytes;
        };
        const bool in_span = vec && o_lo <= w && w + delta >= 0;
        if (in_span && w + U * WE <= o_hi && w + U * WE <= ce && w + U * WE + delta <= NT && tail_ok(U)) {
            const int64_t ab = (w + (int64_t)lane * VE + delta) * E - shift;
            uint4 a[U], x[U];
#pragma unroll
            for (int u = 0; u < U; ++u) a[u] = *reinterpret_cast<const uint4 *>(in + ab + u * 1024);
            if (shift != 0 && lane == kWave - 1) {
#pragma unroll
                for (int u = 0; u < U; ++u) x[u] = *reinterpret_cast<const uint4 *>(in + ab + u * 1024 + 16);
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                uint4 o = a[u];
                if (shift != 0) {
                    uint4 b = shfl_down1(a[u]);
                    if (lane == kWave - 1) b = x[u];
                    o = funnel16(a[u], b, shift);
                }
                store_nt(reinterpret_cast<uint4 *>(out + (w + (int64_t)u * WE + (int64_t)lane * VE) * E), o);
            }
            w += (U - 1) * WE;
            continue;
        }
        if (in_span && w + WE <= o_hi && w + WE <= ce && w + WE + delta <= NT && tail_ok(1)) {
            const int64_t ab = (w + (int64_t)lane * VE + delta) * E - shift;
            const uint4 a = *reinterpret_cast<const uint4 *>(in + ab);
            uint4 o = a;
            if (shift != 0) {
                uint4 b = shfl_down1(a);
                if (lane == kWave - 1) b = *reinterpret_cast<const uint4 *>(in + ab + 16);
                o = funnel16(a, b, shift);
            }
            store_nt(reinterpret_cast<uint4 *>(out + (w + (int64_t)lane * VE) * E), o);
            continue;
        }
        // Element path: every span that meets [w, we).
        int64_t jj = j;
        while (true) {
            sp.ensure(jj);
            const int64_t lo = sp.O(jj), hi = sp.O(jj + 1);
            const int64_t d = sp.S(jj) - lo;
            const int64_t a = lo > w ? lo : w;
            const int64_t b = hi < we ? hi : we;
#pragma unroll
            for (int k = 0; k < VE; ++k) {
                const int64_t p = w + (int64_t)lane * VE + k;
                const int64_t src = p + d;
                if (p >= a && p < b && src >= 0 && src < NT)
                    reinterpret_cast<T *>(out)[p] = reinterpret_cast<const T *>(in)[src];
            }
            if (hi >= we || jj + 1 >= n_kept) break;
            ++jj;
        }
        j = jj;
    }
}

template <typename Spans>
__device__ __forceinline__ void copy_range_col(const CompactCols &cols, int col, Spans &sp,
                                               int64_t n_kept, int64_t NT, int64_t cs, int64_t ce,
                                               int64_t j) {
    const char *in = (const char *)cols.in[col];
    char *out = (char *)cols.out[col];
    const bool vec = cols.vec[col] != 0;
    switch (cols.elem[col]) {
        case 1: copy_range<1>(in, out, vec, sp, n_kept, NT, cs, ce, j); break;
        case 2: copy_range<2>(in, out, vec, sp, n_kept, NT, cs, ce, j); break;
        case 4: copy_range<4>(in, out, vec, sp, n_kept, NT, cs, ce, j); break;
        default: copy_range<8>(in, out, vec, sp, n_kept, NT, cs, ce, j); break;
    }
}

// ---------------------------------------------------------------------------
// Range path
// ---------------------------------------------------------------------------
constexpr int kPT = 256;                  // threads of a copying workgroup
constexpr int kPW = kPT / kWave;          // its waves
constexpr int kCopyU = 4;                 // 16-byte loads in flight per thread in a range copy
constexpr int64_t kRangeMin = 1024;       // tokens of a range when the batch does not fill the chip
constexpr int64_t kRangeLen = 3584;       // tokens of a range when it does
constexpr int64_t kRangeLeast = 2048;     // a range is no shorter than this or the pool's mean trajectory
constexpr int64_t kRangePool = 16384;     // tokens of the pool per range, at most, whatever is expected to be kept
constexpr int64_t kRangeSpans = 2;        // kept trajectories per range, at most, while the chip is not full
constexpr int64_t kWaveCopy = 2048;       // a span part of at most this many bytes is one wave's

// Span length of trajectory i if kept (offsets clamped to [0, NT]), else 0.
// (The flag and both offsets are loaded together: one round trip.)
__device__ __forceinline__ int64_t kept_span(const int64_t *__restrict__ off, const uint8_t *__restrict__ keep,
                                             int64_t i, int64_t NT, int64_t &lo) {
    const bool k = keep[i] != 0;
    const int64_t a = off[i], b = off[i + 1];
    lo = 0;
    if (!k) return -1;
    lo = clamp64(a, 0, NT);
    const int64_t hi = clamp64(b, 0, NT);
    return hi > lo ? hi - lo : 0;
}

// One wave per block of kBlk trajectories: the block partials from the keep
// flags.
template <int kBlk>
__global__ __launch_bounds__(kWave) void compact_partials_kernel(const int64_t *__restrict__ off, int64_t n,
                                                                int64_t NT, const uint8_t *__restrict__ keep,
                                                                PieceParts parts) {
    const int lane = lane_id();
    const int64_t i = (int64_t)blockIdx.x * kBlk + lane;
    int64_t len = 0, lo;
    bool kept = false;
    if (lane < kBlk && i < n) {
        const int64_t k = kept_span(off, keep, i, NT, lo);
        kept = k >= 0;
        len = kept ? k : 0;
    }
    const uint32_t c = (uint32_t)__popcll(ballot(kept));
    const int64_t l = wave_sum_i64(len);
    if (lane == 0) {
        parts.cnt[blockIdx.x] = (int32_t)c;
        parts.len[blockIdx.x] = l;
    }
}

// kThreads threads (t = 0 .. kThreads - 1, whole waves) copy nb bytes from src
// to dst, any alignment of either: aligned 16-byte non-temporal stores, their
// sources as 16-byte loads at whatever byte they start on, kCopyU in flight
// per thread; the fewer than 16 bytes before the first and after the last
// aligned store go out as one unaligned 16-byte store each, which repeats
// bytes of its neighbour. (One- and two-byte columns and columns off 16-byte
// alignment went element by element before: 1024 trajectories, five columns
// of 1 to 8 bytes at odd starts, 138 us, now 26.) The two end stores follow
// the stream: ahead of it, the first wave waits a round trip for them (0.4 us
// of the 50M-token step).
template <int kThreads>
__device__ __forceinline__ void copy_bytes(const char *__restrict__ src, char *__restrict__ dst, int64_t nb, int t) {
    if (nb < 16) {
        if (t < nb) dst[t] = src[t];
        return;
    }
    const int64_t h = (int64_t)(-(uintptr_t)dst & 15);
    const int64_t nv = (nb - h) / 16;
    const char *sv = src + h;
    uint4 *dv = reinterpret_cast<uint4 *>(dst + h);
    int64_t v = t;
    for (; v + (kCopyU - 1) * kThreads < nv; v += kCopyU * kThreads) {
        uint4 x[kCopyU];
#pragma unroll
        for (int u = 0; u < kCopyU; ++u) x[u] = load_a1(sv + (v + u * kThreads) * 16);
#pragma unroll
        for (int u = 0; u < kCopyU; ++u) store_nt(dv + v + u * kThreads, x[u]);
    }
    for (; v < nv; v += kThreads) store_nt(dv + v, load_a1(sv + v * 16));
    if (t == kThreads - 64 && h != 0) store_a1(dst, load_a1(src));
    if (t == kThreads - 63 && h + nv * 16 != nb) store_a1(dst + nb - 16, load_a1(src + nb - 16));
}

// nb < 16 bytes by one thread, any alignment: the two accesses of the largest
// power of two not above nb that cover them, both loaded before either is
// stored. (A byte at a time is nb round trips: 65,536 trajectories of 16 tokens,
// 6553 kept, a one-byte column and two of four 17.2 us, now 13.9.)
template <typename T>
__device__ __forceinline__ void copy_two(const char *__restrict__ src, char *__restrict__ dst, int nb) {
    struct __attribute__((packed)) U { T v; };
    const T a = reinterpret_cast<const U *>(src)->v, b = reinterpret_cast<const U *>(src + nb - sizeof(T))->v;
    reinterpret_cast<U *>(dst)->v = a;
    reinterpret_cast<U *>(dst + nb - sizeof(T))->v = b;
}
__device__ __forceinline__ void copy_under16(const char *__restrict__ src, char *__restrict__ dst, int nb) {
    if (nb >= 8) copy_two<uint64_t>(src, dst, nb);
    else if (nb >= 4) copy_two<uint32_t>(src, dst, nb);
    else if (nb >= 2) copy_two<uint16_t>(src, dst, nb);
    else if (nb == 1) dst[0] = src[0];
}

// A workgroup's part of a span: all its waves together, or a short part by one
// wave, in turn.
__device__ __forceinline__ void copy_part(const char *__restrict__ src, char *__restrict__ dst, int64_t nb, int wv,
                                          int &turn) {
    if (nb > kWaveCopy) copy_bytes<kPT>(src, dst, nb, (int)threadIdx.x);
    else if ((turn++ & (kPW - 1)) == wv) copy_bytes<kWave>(src, dst, nb, lane_id());
}

// Inclusive sums of the block partials x[0 .. nb). kC > 0: kPW * kC * 64 blocks
// at most, kC chunks of 64 per wave, summed once by the workgroup and kept in
// LDS (a barrier); every wave loading all 512 partials of an 8192-trajectory
// pool by itself took 3 to 8 us of a 10 us compaction. kC = 0: at most 64
// blocks, in the registers of every wave; no barrier, 0.8 us of a
// 1024-trajectory step.
template <typename T, int kC>
struct BlockSums {
    static constexpr int kPer = (kC > 0 ? kC : 1) * kWave;      // blocks a wave sums
    struct Smem {
        T sum[kC > 0 ? kPW * kPer : 1];                         // inclusive, within the wave's blocks
        T tot[kPW];
    };
    Smem &sm;
    int64_t start[kPW];                                         // sum before wave w's blocks
    int64_t all;
    T reg;                                                      // kC = 0: the lane's inclusive sum
    T v[kC > 0 ? kC : 1];
    __device__ __forceinline__ explicit BlockSums(Smem &s) : sm(s) {}
    __device__ __forceinline__ void load(const T *__restrict__ x, int64_t nb, int wv) {
#pragma unroll
        for (int c = 0; c < kPer / kWave; ++c) {
            const int64_t b = (kC > 0 ? wv * kPer : 0) + c * kWave + lane_id();
            v[c] = b < nb ? x[b] : (T)0;
        }
    }
    // After load; with kC > 0 a barrier belongs between scan and finish.
    __device__ __forceinline__ void scan(int wv) {
        int64_t run = 0;
#pragma unroll
        for (int c = 0; c < kPer / kWave; ++c) {
            const int64_t incl = run + wave_incl_scan_i64((int64_t)v[c]);
            if constexpr (kC > 0) sm.sum[wv * kPer + c * kWave + lane_id()] = (T)incl;
            else reg = (T)incl;
            run = readlane_i64(incl, kWave - 1);
        }
        all = run;
        if (kC > 0 && lane_id() == 0) sm.tot[wv] = (T)run;
    }
    __device__ __forceinline__ void finish() {
        start[0] = 0;
        if constexpr (kC > 0) {
            all = 0;
#pragma unroll
            for (int w = 0; w < kPW; ++w) {
                start[w] = all;
                all += readlane_i64((int64_t)sm.tot[w], 0);
            }
        }
    }
    // Sum before block b, and the first block whose inclusive sum is above x
    // (x below `all`), with the sum before it: all wave-uniform.
    __device__ __forceinline__ int64_t before(int64_t b) const {
        if constexpr (kC == 0) {
            const int64_t s = readlane_i64((int64_t)reg, b > 0 ? (int)b - 1 : 0);
            return b > 0 ? s : 0;
        }
        int64_t s = b % kPer ? (int64_t)sm.sum[b - 1] : 0;
#pragma unroll
        for (int w = 1; w < kPW; ++w) s += b / kPer == w ? start[w] : 0;
        return s;
    }
    __device__ __forceinline__ int64_t find(int64_t x, int64_t &lo) const {
        int w = 0;
        lo = 0;
        if constexpr (kC > 0) {
#pragma unroll
            for (int k = 1; k < kPW; ++k) {
                if (x >= start[k]) {
                    w = k;
                    lo = start[k];
                }
            }
        }
        const int64_t base = lo;
        int64_t b = w * kPer;
#pragma unroll
        for (int c = 0; c < kPer / kWave; ++c) {
            const int64_t incl = base + (int64_t)(kC > 0 ? sm.sum[kC > 0 ? w * kPer + c * kWave + lane_id() : 0] : reg);
            const uint64_t m = ballot(incl > x);
            const int j = m ? __ffsll((long long)m) - 1 : kWave;
            if (j > 0) lo = readlane_i64(incl, j - 1);
            b += j;
            if (m) break;
        }
        return b;
    }
};

// Workgroups [0, n_idx) write the index outputs (packed offsets, kept ids,
// rejected ids), one block per wave. Then workgroup n_idx + r of grid row col
// copies packed tokens [r S, (r + 1) S) of column col, S = ceil(total / n_rng)
// or `least`, the longer: bound by memory, so the output is cut evenly whatever
// the spans' lengths, finely enough that workgroups ending early leave room for
// others, and by column (the ranges of one column before the next's). Each
// looks its range up in the block partials' sums, then in the spans of the 64
// trajectories from that block on (of the block's own 16, a range of few tokens
// and many blocks takes a round trip a block: 819 of 8192 single tokens, two
// columns, 15.2 us, now 10.4);
// 60 to 64 VGPRs, so that eight workgroups share a CU and one's look-up hides
// under the others' copies. All waves copy a long span part together; parts of
// at most kWaveCopy bytes go to the waves in turn.
// Against whole spans cut into pieces of 16,384 tokens with all columns in one
// workgroup, a fused step: 10M kept tokens in 3 columns 86 -> 67 us, 16.9M in 4
// columns 149 -> 97 us, 16.7M in one column 79 -> 71 us.
template <int kC>
__global__ __launch_bounds__(kPT) void compact_range_kernel(
    const int64_t *__restrict__ off, int64_t n, int64_t NT, const uint8_t *__restrict__ keep,
    PieceParts parts, int64_t nb, int64_t n_idx, int64_t n_rng, int64_t least, CompactCols cols,
    int64_t *__restrict__ offsets_out, int32_t *__restrict__ kept_ids, int64_t *__restrict__ n_kept_tokens,
    int32_t *__restrict__ reject_ids, int64_t budget) {
    __shared__ typename BlockSums<int64_t, kC>::Smem s_len;
    __shared__ typename BlockSums<int32_t, kC>::Smem s_cnt;
    const int lane = lane_id();
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    const int64_t q = blockIdx.x;
    BlockSums<int64_t, kC> L(s_len);
    L.load(parts.len, nb, wv);
    if (q < n_idx) {
        if (blockIdx.y != 0) return;
        BlockSums<int32_t, kC> C(s_cnt);
        C.load(parts.cnt, nb, wv);
        const int64_t b = q * kPW + wv;
        const int64_t i = b * kPieceBlock + lane;
        const bool in = lane < kPieceBlock && i < n;
        int64_t len = 0, lo;
        bool kept = false;
        if (in) {
            const int64_t k = kept_span(off, keep, i, NT, lo);
            kept = k >= 0;
            len = kept ? k : 0;
        }
        L.scan(wv);
        C.scan(wv);
        if (kC > 0) __syncthreads();
        L.finish();
        C.finish();
        if (q == 0 && threadIdx.x == 0) {
            offsets_out[C.all] = L.all;
            *n_kept_tokens = L.all;
        }
        if (b >= nb) return;
        const int64_t rank = C.before(b) + (int64_t)__popcll(ballot(kept) & lanes_below());
        const int64_t dst = L.before(b) + (wave_incl_scan_i64(len) - len);
        if (kept) {
            offsets_out[rank] = dst;
            kept_ids[rank] = (int32_t)i;
        } else if (in && reject_ids) {
            const int64_t rr = i - rank;       // trajectories before i that were rejected
            if (rr < budget) reject_ids[rr] = (int32_t)i;
        }
        return;
    }

    // Copy: packed tokens [x, x1).
    L.scan(wv);
    if (kC > 0) __syncthreads();
    L.finish();
    const int64_t total = L.all < NT ? L.all : NT;   // malformed offsets could overflow the output
    int64_t S = (total + n_rng - 1) / n_rng;
    S = S > least ? S : least;
    S = S < 512 ? (S + 15) / 16 * 16 : (S + 63) / 64 * 64;
    int64_t x = (q - n_idx) * S;
    if (x >= total) return;
    const int64_t x0 = x;
    const int64_t x1 = x0 + S < total ? x0 + S : total;
    const int col = blockIdx.y;
    const int64_t E = cols.elem[col];
    const char *in = (const char *)cols.in[col];
    char *out = (char *)cols.out[col];
    int turn = 0;
    while (x < x1) {
        int64_t lb;
        const int64_t b = L.find(x, lb);
        const int64_t i = b * kPieceBlock + lane;
        int64_t len = 0, lo = 0;
        if (i < n) {
            const int64_t k = kept_span(off, keep, i, NT, lo);
            len = k > 0 ? k : 0;
        }
        const int64_t incl = wave_incl_scan_i64(len);
        const int64_t d = lb + incl - len, nx = lb + readlane_i64(incl, kWave - 1);
        uint64_t m = ballot(len > 0 && d < x1 && d + len > x0);
        while (m) {
            const int j = __ffsll((long long)m) - 1;
            m &= m - 1;
            const int64_t dj = readlane_i64(d, j), lj = readlane_i64(len, j), sj = readlane_i64(lo, j);
            const int64_t a = dj > x0 ? dj : x0;
            const int64_t e = dj + lj < x1 ? dj + lj : x1;
            copy_part(in + (sj + (a - dj)) * E, out + a * E, (e - a) * E, wv, turn);
        }
        if (nx <= x) return;
        x = nx;
    }
}

// Small pools in the filter step: the rank and the range copy in one launch, since a launch costs such a step more than the work
// (the host 3.7 us, the device 3 to 4). Every workgroup ranks all trajectories,
// one per thread, against the keys in LDS (rank_i = #{j : key_j > key_i} +
// #{j < i : key_j == key_i}; of another wave's trajectories all ids lie on one
// side, so one compare decides), scans the kept spans into a table and copies
// its range; workgroup 0 writes the keep flags and index outputs, and joins
// trajectories summed in pieces into their outputs. 64 trajectories, 70K tokens
// 16.4 -> 13.4 us a step.
template <bool kJoin>
__global__ __launch_bounds__(kPT) void rank_compact_small_kernel(
    const double *__restrict__ score, const int64_t *__restrict__ off, int64_t n, int64_t NT, int64_t budget,
    int64_t n_rng, uint8_t *__restrict__ keep, CompactCols cols, int n_cols, int64_t *__restrict__ offsets_out,
    int32_t *__restrict__ kept_ids, int64_t *__restrict__ n_kept_tokens, int32_t *__restrict__ reject_ids,
    ScoreJoin join) {
    static_assert(kSmallMaxN == kPT, "one trajectory per thread");
    __shared__ uint64_t s_key[kPT];
    __shared__ int64_t s_dst[kPT + 1], s_src[kPT];
    __shared__ uint32_t w_cnt[kPW];
    __shared__ int64_t w_len[kPW];
    const int t = threadIdx.x;
    const int wv = __builtin_amdgcn_readfirstlane(t / kWave);
    const bool in = t < n, writer = blockIdx.x == 0 && blockIdx.y == 0;
    double s = 0.0;
    int64_t lo = 0, hi = 0;
    if (in) {
        s = score[t];
        lo = clamp64(off[t], 0, NT);
        hi = clamp64(off[t + 1], 0, NT);
    }
    if (kJoin && in && is_join_mark(s)) s = writer ? write_joined(t, s, join) : joined_score(s, join).score;
    // A number's key is above 0 (-inf's is the smallest), padding is 0.
    const uint64_t key = in ? score_key(s) : 0ull;
    s_key[t] = key;
    __syncthreads();
    uint32_t r = 0;
    const int nw = (int)((n + kWave - 1) / kWave);
    for (int g = 0; g < nw; ++g) {
        const uint64_t *k = s_key + g * kWave;
        if (g == wv) {
            for (int j = 0; j < kWave; ++j) r += (k[j] > key || (k[j] == key && j < lane_id())) ? 1u : 0u;
        } else {
            const uint64_t edge = g < wv ? key - 1 : key;
#pragma unroll 16
            for (int j = 0; j < kWave; ++j) r += k[j] > edge ? 1u : 0u;
        }
    }
    const bool kept = in && (int64_t)r >= budget;
    const int64_t len = kept && hi > lo ? hi - lo : 0;
    uint32_t m;
    int64_t sum;
    const int64_t rank = block_excl_sum_u32<kPW>(kept ? 1u : 0u, m, w_cnt);
    const int64_t dst = block_excl_sum_i64<kPW>(len, sum, w_len);
    if (kept) {
        s_dst[rank] = dst;
        s_src[rank] = lo;
    }
    if (t == 0) s_dst[m] = sum;
    if (writer && in) {
        keep[t] = kept ? 1 : 0;
        if (kept) {
            offsets_out[rank] = dst;
            kept_ids[rank] = t;
        } else if (t - rank < budget) {
            reject_ids[t - rank] = t;
        }
    }
    if (writer && t == 0) {
        offsets_out[m] = sum;
        *n_kept_tokens = sum;
    }
    __syncthreads();
    const int64_t total = sum < NT ? sum : NT;   // malformed offsets could overflow the output
    const int64_t S = ((total + n_rng - 1) / n_rng + 63) / 64 * 64;
    const int64_t x0 = (int64_t)blockIdx.x * S;
    if (n_cols == 0 || x0 >= total) return;
    const int64_t x1 = x0 + S < total ? x0 + S : total;
    const int col = blockIdx.y;
    const int64_t E = cols.elem[col];
    const char *in_c = (const char *)cols.in[col];
    char *out_c = (char *)cols.out[col];
    // The last span starting at or before x0.
    int j = 0;
    for (int step = kPT / 2; step > 0; step >>= 1)
        if (j + step < (int)m && readlane_i64(s_dst[j + step], 0) <= x0) j += step;
    int turn = 0;
    for (; j < (int)m; ++j) {
        const int64_t d = readlane_i64(s_dst[j], 0), d1 = readlane_i64(s_dst[j + 1], 0);
        if (d >= x1) return;
        const int64_t a = d > x0 ? d : x0, e = d1 < x1 ? d1 : x1;
        if (a < e) copy_part(in_c + (readlane_i64(s_src[j], 0) + (a - d)) * E, out_c + a * E, (e - a) * E, wv, turn);
    }
}

// ---------------------------------------------------------------------------
// Wide path: blocks of kWideBlock trajectories, the copy split by merge path
// ---------------------------------------------------------------------------
// The block partials come in two levels: per block (kept count and tokens)
// and per group of kGroupBlocks blocks (their sums), so that a workgroup
// finds any block's packed position from at most kWideMaxGroups group sums
// and the kGroupBlocks - 1 blocks before it in its group, with wave
// reductions and no scan over all blocks.
//
// The packed output is split evenly by a merge path over the cost (kept
// tokens + kBlockCost per block): workgroup q copies the kept tokens of cost
// range [q S, (q + 1) S), S = ceil(total cost / grid), which holds at most
// S / kBlockCost + 2 blocks, four blocks (one per wave) at a time. Then wave w
// of workgroup q writes the index outputs of block q + w * grid.
constexpr int64_t kBlockCost = 2048;
constexpr int kSpanT = kPT;               // spans in one copy table: four blocks of one wave each
constexpr int kSpanU = 8;                 // 16-byte loads in flight per thread in a span copy
struct SpanTable {
    int32_t start[kSpanT];       // first slot of each span
    int64_t dst[kSpanT];         // byte offset of each span's first slot
    int64_t src[kSpanT];         // byte offset of its source
};

// The span holding slot g: the last span whose first slot is <= g.
__device__ __forceinline__ int span_find(const SpanTable &tb, int32_t g) {
    int j = 0;
#pragma unroll
    for (int step = kSpanT / 2; step > 0; step >>= 1) j = tb.start[j + step] <= g ? j + step : j;
    return j;
}

// Thread t brings span t's destination range [a, b) in elements and its shift
// del (source - destination). The slots are the aligned 16-byte vectors of
// the destination, their sources 16-byte loads at whatever byte they start
// on. Each thread copies the fewer than 16 bytes at each end of its own range
// as one unaligned vector that repeats bytes of its neighbour, or a range
// shorter than a vector by itself. Their loads go first, while the table is
// built: 65,536 trajectories of 700 tokens, half kept, 41.6 -> 41.0 us; of 100
// tokens, one-byte column and two of four 25.2 -> 21.7.
__device__ __forceinline__ void copy_spans_col(const CompactCols &cols, int col, int64_t a, int64_t b, int64_t del,
                                               SpanTable &tb, uint32_t *wsum) {
    const int64_t E = cols.elem[col];
    // Offsets from the last 16-byte boundary at or before the column's start.
    const int64_t ph = (int64_t)((uintptr_t)cols.out[col] & 15);
    const char *src = (const char *)cols.in[col] - ph;
    char *dst = (char *)cols.out[col] - ph;
    const int t = threadIdx.x;
    const int64_t a0 = a * E + ph, b0 = b * E + ph, dl = del * E;
    int64_t v0 = (a0 + 15) / 16 * 16, v1 = b0 / 16 * 16;
    if (v1 < v0) v0 = v1 = b0;
    uint4 h, e;
    if (b0 - a0 >= 16) {
        if (a0 < v0) h = load_a1(src + a0 + dl);
        if (v1 < b0) e = load_a1(src + b0 - 16 + dl);
    } else {
        copy_under16(src + a0 + dl, dst + a0, (int)(b0 - a0));
    }
    // (The sum's barriers also end the reading of the previous table.)
    uint32_t tot;
    const uint32_t ex = block_excl_sum_u32<kPW>((uint32_t)((v1 - v0) / 16), tot, wsum);
    if (tot != 0) {                            // there are slots
        tb.start[t] = (int32_t)ex;
        tb.dst[t] = v0;
        tb.src[t] = v0 + dl;
        __syncthreads();
        const int32_t total = (int32_t)tot;
        for (int32_t g0 = t; g0 < total; g0 += kSpanU * kPT) {
            uint4 x[kSpanU];
#pragma unroll
            for (int u = 0; u < kSpanU; ++u) {
                const int32_t g = g0 + u * kPT;
                if (g < total) {
                    const int j = span_find(tb, g);
                    x[u] = load_a1(src + tb.src[j] + (int64_t)(g - tb.start[j]) * 16);
                }
            }
#pragma unroll
            for (int u = 0; u < kSpanU; ++u) {
                const int32_t g = g0 + u * kPT;
                if (g < total) {
                    const int j = span_find(tb, g);
                    store_nt(reinterpret_cast<uint4 *>(dst + tb.dst[j] + (int64_t)(g - tb.start[j]) * 16), x[u]);
                }
            }
        }
    }
    if (b0 - a0 >= 16) {
        if (a0 < v0) store_a1(dst + a0, h);
        if (v1 < b0) store_a1(dst + b0 - 16, e);
    }
}

// One workgroup of 1024 threads per kGroupBlocks blocks of kWideBlock
// trajectories (one wave each): the block partials from the keep flags and
// the group's sums.
__global__ __launch_bounds__(kWideBlock * kGroupBlocks) void compact_partials_wide_kernel(
    const int64_t *__restrict__ off, int64_t n, int64_t NT, const uint8_t *__restrict__ keep, PieceParts parts) {
    static_assert(kWideBlock == kWave, "a wide block is one wave");
    __shared__ uint32_t sc[kGroupBlocks];
    __shared__ int64_t sl[kGroupBlocks];
    const int lane = lane_id(), w = threadIdx.x / kWave;
    const int64_t b = (int64_t)blockIdx.x * kGroupBlocks + w;
    const int64_t i = b * kWideBlock + lane;
    int64_t len = 0, lo;
    bool kept = false;
    if (i < n) {
        const int64_t k = kept_span(off, keep, i, NT, lo);
        kept = k >= 0;
        len = kept ? k : 0;
    }
    const uint32_t c = (uint32_t)__popcll(ballot(kept));
    const int64_t l = wave_sum_i64(len);
    if (lane == 0) {
        if (b * kWideBlock < n) {
            parts.cnt[b] = (int32_t)c;
            parts.len[b] = l;
        }
        sc[w] = c;
        sl[w] = l;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t gc = 0;
        int64_t gl = 0;
        for (int k = 0; k < kGroupBlocks; ++k) {
            gc += sc[k];
            gl += sl[k];
        }
        parts.gcnt[blockIdx.x] = (int32_t)gc;
        parts.glen[blockIdx.x] = gl;
    }
}

// nb blocks in ng = ceil(nb / kGroupBlocks) <= kWideMaxGroups groups;
// 4 * grid >= nb.
__global__ __launch_bounds__(kPT) void compact_wide_kernel(
    const int64_t *__restrict__ off, int64_t n, int64_t NT, const uint8_t *__restrict__ keep,
    PieceParts parts, int64_t nb, CompactCols cols, int n_cols, int64_t *__restrict__ offsets_out,
    int32_t *__restrict__ kept_ids, int64_t *__restrict__ n_kept_tokens, int32_t *__restrict__ reject_ids,
    int64_t budget) {
    static_assert(kWideBlock == kWave, "a wide block is one wave");
    static_assert(kWideMaxGroups == 4 * kWave, "group sums: four per lane of one wave");
    __shared__ int64_t s_gl[kWideMaxGroups + 1];   // kept tokens before each group; [kWideMaxGroups] = total
    __shared__ uint32_t s_gc[kWideMaxGroups + 1];  // kept trajectories before each group
    __shared__ int64_t s_cut[6];                   // b0, b1, x0, x1
    __shared__ uint32_t wsum[kPW];
    __shared__ SpanTable tb;
    const int t = threadIdx.x, w = t / kWave, lane = lane_id();
    const int64_t q = blockIdx.x, G = gridDim.x;
    const int64_t ng = (nb + kGroupBlocks - 1) / kGroupBlocks;

    // The block `b`'s kept count and tokens before it inside its group: the
    // wave's lanes below kGroupBlocks hold the group's earlier blocks.
    auto in_group = [&](int64_t b, uint32_t &c, int64_t &l) {
        const int64_t j = b / kGroupBlocks * kGroupBlocks + lane;
        c = 0u;
        l = 0;
        if (lane < kGroupBlocks && j < b) {
            c = (uint32_t)parts.cnt[j];
            l = parts.len[j];
        }
    };

    // 0. The index block of this wave: its spans and its group's earlier
    //    partials, loaded with the group sums (one round trip).
    const int64_t ib = q + (int64_t)w * G;
    int64_t i_lo = 0, i_len = -1;
    uint32_t i_c = 0u;
    int64_t i_l = 0;
    if (ib < nb) {
        const int64_t i = ib * kWideBlock + lane;
        if (i < n) {
            const uint8_t kf = keep[i];
            const int64_t a = off[i], b = off[i + 1];
            if (kf != 0) {
                i_lo = clamp64(a, 0, NT);
                const int64_t hi = clamp64(b, 0, NT);
                i_len = hi > i_lo ? hi - i_lo : 0;
            }
        }
        in_group(ib, i_c, i_l);
    }

    // 1. Exclusive prefixes of the group sums (wave 0, four groups per lane).
    if (w == 0) {
        uint32_t c4[4];
        int64_t l4[4];
        uint32_t cs = 0u;
        int64_t ls = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int64_t g = (int64_t)lane * 4 + k;
            c4[k] = g < ng ? (uint32_t)parts.gcnt[g] : 0u;
            l4[k] = g < ng ? parts.glen[g] : 0;
            cs += c4[k];
            ls += l4[k];
        }
        uint32_t ce = wave_incl_scan_u32(cs) - cs;
        int64_t le = wave_incl_scan_i64(ls) - ls;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            s_gc[lane * 4 + k] = ce;
            s_gl[lane * 4 + k] = le;
            ce += c4[k];
            le += l4[k];
        }
        if (lane == kWave - 1) {
            s_gc[kWideMaxGroups] = ce;
            s_gl[kWideMaxGroups] = le;
        }
    }
    __syncthreads();
    const int64_t tot_l = s_gl[kWideMaxGroups];

    // 2. Copy the kept tokens of cost range [q S, (q + 1) S). Wave 0 finds the
    //    blocks holding costs c0, c1 - 1 and c1: per cost, a binary search over
    //    the groups' cost starts, then lanes 16u .. 16u + 15 scan that group's
    //    block lengths (row u of the wave).
    const int64_t T = tot_l + kBlockCost * nb;
    const int64_t S = (T + G - 1) / G;
    const int64_t c0 = q * S;
    if (n_cols > 0 && nb > 0 && c0 < T) {
        const int64_t c1 = (c0 + S < T) ? c0 + S : T;
        if (w == 0) {
            const int u = lane / kGroupBlocks, r = lane % kGroupBlocks;
            const int64_t key = u == 0 ? c0 : (u == 1 ? c1 - 1 : c1);
            int64_t lo = 0, hi = ng;                // last group whose cost starts at or before key
            while (hi - lo > 1) {
                const int64_t mid = (lo + hi) / 2;
                if (s_gl[mid] + kBlockCost * kGroupBlocks * mid <= key) lo = mid;
                else hi = mid;
            }
            const int64_t j = lo * kGroupBlocks + r;
            const int64_t len = (u < 3 && j < nb) ? parts.len[j] : 0;
            const int64_t before = s_gl[lo] + (row_incl_scan_i64(len) - len);
            const int64_t cst = before + kBlockCost * j;   // cost start of block j
            const bool ok = u < 3 && j < nb && cst <= key;
            const uint64_t m = ballot(ok);
            const uint32_t row = (uint32_t)(m >> (16 * u)) & 0xffffu;
            const bool last = ok && (row >> (r + 1)) == 0u;
            if (last) {
                if (u == 0) s_cut[0] = j;
                if (u == 1) s_cut[1] = j;
                const int64_t rr = key - cst - kBlockCost;
                const int64_t x = before + (rr < 0 ? 0 : (rr > len ? len : rr));
                if (u == 0) s_cut[2] = x;
                if (u == 2) s_cut[3] = x;
            }
        }
        __syncthreads();
        const int64_t b0 = s_cut[0], b1 = s_cut[1], x0 = s_cut[2], x1 = s_cut[3];
        for (int64_t bg = b0; x0 < x1 && bg <= b1; bg += kPW) {
            // Wave w: block bg + w, lane j its trajectory j; the part of its
            // kept span inside [x0, x1).
            const int64_t b = bg + w;
            int64_t a = 0, e = 0, del = 0;
            if (b <= b1) {
                const int64_t i = b * kWideBlock + lane;
                int64_t len = 0, lo_i = 0;
                if (i < n) {
                    const int64_t k = kept_span(off, keep, i, NT, lo_i);
                    len = k > 0 ? k : 0;
                }
                uint32_t gc;
                int64_t gl;
                in_group(b, gc, gl);
                const int64_t lb = s_gl[b / kGroupBlocks] + wave_sum_i64(gl);
                const int64_t dst = lb + (wave_incl_scan_i64(len) - len);
                const int64_t s0 = dst > x0 ? dst : x0;
                const int64_t s1 = (dst + len < x1) ? dst + len : x1;
                if (s1 > s0) {
                    a = s0;
                    e = s1 < NT ? s1 : NT;             // overlapping (malformed) offsets overflow the output
                    if (a > e) a = e;
                    del = lo_i - dst;
                }
            }
            for (int col = 0; col < n_cols; ++col) copy_spans_col(cols, col, a, e, del, tb, wsum);
        }
    }

    // 3. Index outputs of block ib (after the copy: their stores would hold
    //    up the copy's first loads, one counter covering both).
    if (q == 0 && t == 0) {
        offsets_out[s_gc[kWideMaxGroups]] = tot_l;
        *n_kept_tokens = tot_l;
    }
    if (ib < nb) {
        const int64_t i = ib * kWideBlock + lane;
        const bool kept = i_len >= 0;
        const int64_t len = kept ? i_len : 0;
        const int64_t g = ib / kGroupBlocks;
        const int64_t cb = (int64_t)s_gc[g] + (int64_t)wave_sum_u64((uint64_t)i_c);
        const int64_t lb = s_gl[g] + wave_sum_i64(i_l);
        const int64_t rank = cb + (int64_t)__popcll(ballot(kept) & lanes_below());
        const int64_t dst = lb + (wave_incl_scan_i64(len) - len);
        if (kept) {
            offsets_out[rank] = dst;
            kept_ids[rank] = (int32_t)i;
        } else if (i < n && reject_ids) {
            const int64_t rr = i - rank;           // trajectories before i that were rejected
            if (rr < budget) reject_ids[rr] = (int32_t)i;
        }
    }
}

// ---------------------------------------------------------------------------
// Scan path
// ---------------------------------------------------------------------------
// hdr[0] = n_kept, hdr[1] = min(total kept tokens, n_tokens)
__global__ __launch_bounds__(kT) void compact_scan_kernel(
    const int64_t *__restrict__ off, int64_t n, int64_t NT, const uint8_t *__restrict__ keep,
    int64_t *__restrict__ offsets_out, int32_t *__restrict__ kept_ids,
    int64_t *__restrict__ n_kept_tokens, int64_t *__restrict__ kept_src,
    int32_t *__restrict__ chunk_first, int64_t map_cap, int64_t *__restrict__ hdr) {
    __shared__ uint32_t wcnt[kNW];
    __shared__ int64_t wlen[kNW];
    int64_t run_cnt = 0, run_len = 0;
    for (int64_t base = 0; base < n; base += kT) {
        const int64_t i = base + threadIdx.x;
        const bool in = i < n;
        const bool k = in && keep[i] != 0;
        int64_t lo = 0, len = 0;
        if (k) {
            lo = clamp64(off[i], 0, NT);
            const int64_t hi = clamp64(off[i + 1], 0, NT);
            len = hi > lo ? hi - lo : 0;
        }
        uint32_t tc;
        const uint32_t r = block_excl_sum_u32<kNW>(k ? 1u : 0u, tc, wcnt);
        int64_t tl;
        const int64_t d = block_excl_sum_i64<kNW>(len, tl, wlen);
        if (k) {
            const int64_t rank = run_cnt + r;
            const int64_t dst = run_len + d;
            offsets_out[rank] = dst;
            kept_ids[rank] = (int32_t)i;
            kept_src[rank] = lo;
            int64_t end = dst + len;
            if (end > NT) end = NT;
            for (int64_t c = (dst + kCopyChunk - 1) / kCopyChunk; c * kCopyChunk < end && c < map_cap; ++c)
                chunk_first[c] = (int32_t)rank;
        }
        run_cnt += tc;
        run_len += tl;
    }
    if (threadIdx.x == 0) {
        offsets_out[run_cnt] = run_len;
        *n_kept_tokens = run_len;
        hdr[0] = run_cnt;
        hdr[1] = run_len < NT ? run_len : NT;
    }
}

__global__ __launch_bounds__(256) void compact_copy_kernel(
    CompactCols cols, const int64_t *__restrict__ oo, const int64_t *__restrict__ ss,
    const int32_t *__restrict__ chunk_first, const int64_t *__restrict__ hdr, int64_t NT) {
    const int col = blockIdx.y;
    const int64_t n_kept = hdr[0];
    const int64_t total = hdr[1];
    if (n_kept <= 0) return;
    const int64_t n_chunks = (total + kCopyChunk - 1) / kCopyChunk;
    const int64_t waves = (int64_t)gridDim.x * (blockDim.x / kWave);
    for (int64_t c = (int64_t)blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave; c < n_chunks; c += waves) {
        const int64_t cs = c * kCopyChunk;
        const int64_t ce = (cs + kCopyChunk < total) ? cs + kCopyChunk : total;
        const int64_t j = clamp64(chunk_first[c], 0, n_kept - 1);
        GlobalSpans sp{oo, ss, n_kept, 0, 0, 0};
        sp.load(j);
        copy_range_col(cols, col, sp, n_kept, NT, cs, ce, j);
    }
}

}  // namespace

int64_t map_capacity(int64_t n_tokens) { return (n_tokens + kCopyChunk - 1) / kCopyChunk + 1; }

CompactWs compact_ws_carve(void *ws, int64_t n, int64_t n_tokens) {
    const size_t nb = (size_t)piece_blocks(n);
    char *p = (char *)ws;
    CompactWs w;
    w.hdr = (int64_t *)p;          p += 256;
    w.kept_src = (int64_t *)p;     p += align256((size_t)n * 8);
    w.chunk_first = (int32_t *)p;  p += align256((size_t)map_capacity(n_tokens) * 4);
    w.parts.cnt = (int32_t *)p;    p += align256(nb * 4);
    w.parts.len = (int64_t *)p;    p += align256(nb * 8);
    p += align256(nb * 4);         // spare: keeps the workspace size that callers know
    const size_t ng = (size_t)wide_groups(n);
    w.parts.gcnt = (int32_t *)p;   p += align256(ng * 4);
    w.parts.glen = (int64_t *)p;
    return w;
}

size_t compact_ws_bytes(int64_t n, int64_t n_tokens) {
    const size_t nb = (size_t)piece_blocks(n);
    const size_t ng = (size_t)wide_groups(n);
    return 256 + align256((size_t)n * 8) + align256((size_t)map_capacity(n_tokens) * 4) +
           align256(nb * 4) * 2 + align256(nb * 8) + align256(ng * 4) + align256(ng * 8);
}

bool compact_piece_ok(int64_t n, int64_t n_tokens) {
    return n <= kPieceMaxN && n_tokens < kPartsMaxTokens;
}

bool compact_wide_ok(int64_t n, int64_t n_tokens) {
    return n <= kWideMaxN && n_tokens < kPartsMaxTokens;
}

hipError_t launch_compact_partials(const int64_t *offsets, int64_t n, int64_t n_tokens,
                                   const uint8_t *keep, const PieceParts &parts, hipStream_t stream,
                                   int blk) {
    if (n == 0) return hipSuccess;
    if (blk == kWideBlock)
        return launch(-1, compact_partials_wide_kernel,
                      dim3((unsigned)((n + kWideBlock * kGroupBlocks - 1) / (kWideBlock * kGroupBlocks))),
                      dim3(kWideBlock * kGroupBlocks), stream, offsets, n, n_tokens, keep, parts);
    return launch(-1, compact_partials_kernel<kPieceBlock>, dim3((unsigned)piece_blocks(n)), dim3(kWave), stream,
                  offsets, n, n_tokens, keep, parts);
}

// Ranges per column. max_kept / n of the tokens is the expected batch: as many
// ranges as fill the chip once (8 workgroups per CU over all columns) while they
// hold kRangeMin tokens, up to 12 per CU and column while they hold kRangeLen.
// Finer ranges even out the workgroups' end times, but each pays its look-up: at
// 4870 trajectories of 620 tokens and four columns, 2040 workgroups take 2 us
// less than 3500; at 10M kept tokens and three columns, 2436 to 3072 ranges of a
// column take 2 us less than 683 and 3 us less than 4096.
// The survivors need not be of mean length, and spans of a few tokens cost a
// round trip each and not their bytes, so the expected tokens do not decide
// alone. One range per kRangePool tokens of the pool: 4 survivors of 400,000
// tokens among 8192 trajectories, a step of 143 us with the 5 ranges of the
// expected tokens, 35 us with these. One range per kRangeSpans survivors: 300
// trajectories of 20 tokens, 100 kept, 46 us with 1 range, 13 us with 50.
static int64_t range_count(int64_t n, int64_t n_tokens, int n_cols, int64_t max_kept) {
    const int64_t cus = resident_waves() / 16;
    const int64_t kept = max_kept < 0 ? 0 : std::min(max_kept, n);
    const int64_t est = expected_kept(n, n_tokens, kept);
    const int64_t want = std::max({est / kRangeMin, n_tokens / kRangePool, kept / kRangeSpans});
    const int64_t fill = std::min(want, cus * 8 / n_cols);
    const int64_t fine = std::min(est / kRangeLen, cus * 12);
    return std::max<int64_t>(std::max(fill, fine), 1);
}

// Least tokens of a range, where fewer are kept than the count above allows for
// (pace_compact cannot know): a range is a look-up, so it holds a mean
// trajectory or kRangeLeast tokens. 819 of 8192 trajectories of 2000 tokens kept,
// one column: 15.1 us in 3072 ranges, 9.5 in 820.
static int64_t range_least(int64_t n, int64_t n_tokens) {
    return n > 0 ? std::min(kRangeLeast, n_tokens / n) : kRangeLeast;
}

hipError_t launch_rank_compact_small(const double *score, const int64_t *offsets, int64_t n, int64_t n_tokens,
                                     int64_t budget, uint8_t *keep, const CompactCols &cols, int n_cols,
                                     int64_t *offsets_out, int32_t *kept_ids, int64_t *n_kept_tokens,
                                     int32_t *reject_ids, hipStream_t stream, const ScoreJoin &join) {
    if (n > kSmallMaxN) return hipErrorInvalidValue;
    // As many ranges as range_count has for such batches (few columns and tokens
    // by small_step_ok): 200 trajectories of 20 tokens, 66 kept, 33 us a step
    // with the one range of the expected tokens, 13.5 with 33.
    const int64_t n_rng = n_cols > 0 ? range_count(n, n_tokens, n_cols, n - budget) : 1;
    const dim3 grid((unsigned)n_rng, (unsigned)(n_cols > 0 ? n_cols : 1));
    if (join.cap)
        return launch(kPhaseCompact, rank_compact_small_kernel<true>, grid, dim3(kPT), stream,
                      (const double *)join.ws.traj, offsets, n, n_tokens, budget, n_rng, keep, cols, n_cols, offsets_out,
                      kept_ids, n_kept_tokens, reject_ids, join);
    return launch(kPhaseCompact, rank_compact_small_kernel<false>, grid, dim3(kPT), stream, score, offsets, n, n_tokens,
                  budget, n_rng, keep, cols, n_cols, offsets_out, kept_ids, n_kept_tokens, reject_ids, join);
}

hipError_t launch_compact_pieces(const int64_t *offsets, int64_t n, int64_t n_tokens, const uint8_t *keep,
                                 const PieceParts &parts, const CompactCols &cols, int n_cols,
                                 int64_t *offsets_out, int32_t *kept_ids, int64_t *n_kept_tokens,
                                 int32_t *reject_ids, int64_t budget, int64_t max_kept,
                                 hipStream_t stream, int blk) {
    const int64_t nb = (n + blk - 1) / blk;
    if (blk == kPieceBlock) {
        if (nb > 8 * kWave) return hipErrorInvalidValue;
        const int64_t n_idx = nb > 0 ? (nb + kPW - 1) / kPW : 1;
        const int64_t n_rng = n_cols > 0 ? range_count(n, n_tokens, n_cols, max_kept) : 0;
        const dim3 grid((unsigned)(n_idx + n_rng), (unsigned)(n_cols > 0 ? n_cols : 1));
#define PACE_RANGES(P)                                                                                          \
    return launch(kPhaseCompact, compact_range_kernel<P>, grid, dim3(kPT), stream, offsets, n, n_tokens, keep,  \
                  parts, nb, n_idx, n_rng, range_least(n, n_tokens), cols, offsets_out, kept_ids, n_kept_tokens, \
                  reject_ids, budget)
        if (nb <= kWave) PACE_RANGES(0);
        if (nb <= 4 * kWave) PACE_RANGES(1);
        PACE_RANGES(2);
#undef PACE_RANGES
    }
    if (blk != kWideBlock || (nb + kGroupBlocks - 1) / kGroupBlocks > kWideMaxGroups) return hipErrorInvalidValue;
    // Every workgroup indexes up to four blocks and copies an even share of
    // the output: one resident round (four per CU).
    int64_t wgs = (nb + kPW - 1) / kPW;
    if (wgs < resident_waves() / 16 * 4) wgs = resident_waves() / 16 * 4;
    if (wgs < 1) wgs = 1;
    return launch(kPhaseCompact, compact_wide_kernel, dim3((unsigned)wgs), dim3(kPT), stream, offsets, n, n_tokens,
                  keep, parts, nb, cols, n_cols, offsets_out, kept_ids, n_kept_tokens, reject_ids, budget);
}

hipError_t launch_compact_copy(const CompactCols &cols, int n_cols, int64_t n_tokens,
                               const int64_t *offsets_out, const CompactWs &w, hipStream_t stream) {
    if (n_cols == 0 || n_tokens == 0) return hipSuccess;
    const int64_t max_chunks = (n_tokens + kCopyChunk - 1) / kCopyChunk;
    int64_t blocks = (max_chunks + 3) / 4;
    if (blocks > 1024) blocks = 1024;
    if (blocks < 1) blocks = 1;
    dim3 grid((unsigned)blocks, (unsigned)n_cols);
    return launch(kPhaseCompact, compact_copy_kernel, grid, dim3(256), stream, cols, offsets_out,
                  w.kept_src, w.chunk_first, w.hdr, n_tokens);
}

hipError_t launch_compact(const int64_t *offsets, int64_t n, int64_t n_tokens, const uint8_t *keep,
                          const CompactCols &cols, int n_cols, int64_t *offsets_out,
                          int32_t *kept_ids, int64_t *n_kept_tokens, void *ws, hipStream_t stream) {
    CompactWs w = compact_ws_carve(ws, n, n_tokens);
    if (compact_piece_ok(n, n_tokens) || compact_wide_ok(n, n_tokens)) {
        const int blk = compact_piece_ok(n, n_tokens) ? kPieceBlock : kWideBlock;
        hipError_t e = launch_compact_partials(offsets, n, n_tokens, keep, w.parts, stream, blk);
        if (e != hipSuccess) return e;
        return launch_compact_pieces(offsets, n, n_tokens, keep, w.parts, cols, n_cols, offsets_out,
                                     kept_ids, n_kept_tokens, nullptr, 0, n, stream, blk);
    }
    compact_scan_kernel<<<1, kT, 0, stream>>>(offsets, n, n_tokens, keep, offsets_out, kept_ids,
                                             n_kept_tokens, w.kept_src, w.chunk_first,
                                             map_capacity(n_tokens), w.hdr);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch_compact_copy(cols, n_cols, n_tokens, offsets_out, w, stream);
}

}  // namespace pace

// pace_filter_step: the whole filter step (Algorithm 1, trainer side) on
// one stream, every phase spread over the whole device:
//
//   1. score_traj     (score_traj.hip) every tag read once, one workgroup per
//                                    trajectory: S, T and the score
//   2. rank           (select.hip)   exact rank by counting -> keep flags,
//                                    plus per-block kept counts and tokens;
//                                    joins trajectories summed in pieces
//   3. compact_range  (compact.hip)  one wave per block writes the packed
//                                    offsets, kept ids and rejected ids; one
//                                    workgroup per range of the packed output
//                                    and column copies it
//
// The same results as pace_score, pace_budget, pace_select and pace_compact
// called in sequence, in three launches; in two for small pools
// (2 and 3 as one kernel, rank_compact_small in compact.hip). Pools beyond the rank kernel's limit
// (8192 trajectories) take the selection spread over the chip instead of the
// rank (select_wide.hip): the scores by trajectory or, for short ones, by
// chunks (score.hip: score_reduce, score_finalize), with per-group key extremes
// and the level-0 histogram cleared by the second of their kernels; then
// cut_hist, and classify, where every workgroup finds the cut and writes keep
// flags, the partials of blocks of 64 trajectories and their group sums; and
// compact_wide (an even merge-path split of the packed output). Pools beyond
// that path's limit use the separate calls' kernels.
#include "device_util.hpp"
#include "kernels.hpp"

namespace pace {

size_t filter_step_ws_bytes(int64_t n, int64_t n_tokens) {
    return align256(score_ws_bytes(n, n_tokens)) + align256(compact_ws_bytes(n, n_tokens)) +
           align256(select_ws_bytes(n));
}

hipError_t launch_filter_step(const int32_t *tags, const int64_t *offsets, int64_t n, int64_t n_tokens,
                              const int32_t *completion, int32_t V, const double *prefix,
                              const double *window, int64_t W, bool use_prefix, double w_wait,
                              int gamma, int64_t budget, double *score, int64_t *gen_sum,
                              int64_t *gen_count, uint8_t *keep, int32_t *reject_ids,
                              const CompactCols &cols, int n_cols, int64_t *offsets_out,
                              int32_t *kept_ids, int64_t *n_kept_tokens, void *ws,
                              hipStream_t stream) {
    char *p = (char *)ws;
    const ScoreWorkspace sws = score_ws_carve(p, n, n_tokens);
    p += align256(score_ws_bytes(n, n_tokens));
    void *cws_base = p;
    p += align256(compact_ws_bytes(n, n_tokens));
    void *sel_ws = p;

    const bool rank_path = n <= kRankMaxN && compact_piece_ok(n, n_tokens);
    const bool wide_path = !rank_path && compact_wide_ok(n, n_tokens);
    const WideWs ww = wide_ws_carve(sel_ws, n);
    const ScoreArgs sa{offsets, n, n_tokens, completion, V, use_prefix ? 1 : 0, gamma, prefix, window, W, w_wait,
                       score, gen_sum, gen_count};
    ScoreJoin join{};
    hipError_t e;
    if (rank_path) {
        e = launch_score_unjoined(tags, sa, sws, stream, &join);
    } else if (wide_path && score_by_traj(n, n_tokens)) {
        e = launch_score_traj(tags, sa, sws, stream);
        if (e == hipSuccess) e = launch_score_join(sa, sws, stream, ww.mmin, ww.mmax, ww.hist);
    } else if (wide_path) {
        int64_t chunk_len = 0;
        e = launch_score_reduce(tags, offsets, n, n_tokens, V, sws, stream, &chunk_len);
        if (e == hipSuccess)
            e = launch_score_finalize(offsets, n, n_tokens, completion, V, prefix, window, W, use_prefix, w_wait, gamma,
                                      chunk_len, score, gen_sum, gen_count, sws, stream, ww.mmin, ww.mmax, ww.hist);
    } else {
        e = launch_score(tags, sa, sws, stream);
    }
    if (e != hipSuccess) return e;
    if (wide_path) {
        const CompactWs cw = compact_ws_carve(cws_base, n, n_tokens);
        e = launch_wide_cut(score, n, budget, ww, stream);
        if (e != hipSuccess) return e;
        e = launch_classify(score, offsets, n, n_tokens, budget, ww, keep, cw.parts, stream);
        if (e != hipSuccess) return e;
        const int64_t n_kept = n - (budget < n ? budget : n);
        return launch_compact_pieces(offsets, n, n_tokens, keep, cw.parts, cols, n_cols, offsets_out,
                                     kept_ids, n_kept_tokens, reject_ids, budget, n_kept, stream, kWideBlock);
    }
    if (rank_path && small_step_ok(n, n_tokens, n_cols, budget))
        return launch_rank_compact_small(score, offsets, n, n_tokens, budget, keep, cols, n_cols, offsets_out, kept_ids,
                                         n_kept_tokens, reject_ids, stream, join);
    if (rank_path) {
        const CompactWs cw = compact_ws_carve(cws_base, n, n_tokens);
        e = launch_rank(score, n, budget, keep, offsets, n_tokens, cw.parts, stream, join);
        if (e != hipSuccess) return e;
        // The rank rejects exactly min(budget, n) trajectories.
        const int64_t n_kept = n - (budget < n ? budget : n);
        return launch_compact_pieces(offsets, n, n_tokens, keep, cw.parts, cols, n_cols, offsets_out,
                                     kept_ids, n_kept_tokens, reject_ids, budget, n_kept, stream);
    }
    e = launch_select(score, n, budget, keep, reject_ids, sel_ws, stream);
    if (e != hipSuccess) return e;
    return launch_compact(offsets, n, n_tokens, keep, cols, n_cols, offsets_out, kept_ids,
                          n_kept_tokens, cws_base, stream);
}

}  // namespace pace

"""The compaction's cut into ranges where the survivors are not of the pool's mean
length: a few long ones, many of a few tokens, and runs of rejected blocks, on
both sides of the sizes where the look-up of the block sums changes (1024 and
4096 trajectories) and of the small steps (256); and that such batches keep the
chip busy, by the copy kernel's own time."""
import sys

import numpy as np
import pytest

import oracle
import poolgen
from tests.test_gpu_parity import D, H, assert_same, gpu_step, oracle_step

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def say(msg):
    sys.stdout.write("[gpu] %s\n" % msg)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def pace():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2609_36830_amd as pace
    return pace


def _lengths(kind, n):
    rng = np.random.default_rng(n)
    if kind == "short":
        return rng.integers(0, 24, n)
    L = rng.integers(0, 90, n)
    L[[0, n // 3, n // 3 + 1, n - 1]] = [30011, 64000, 2049, 17001]
    return L


def _fresh(pool, kept):
    """The `kept` longest trajectories consumed at their own version, the others
    a version late: those survive."""
    top = np.sort(np.argsort(-np.diff(pool.offsets), kind="stable")[:kept])
    pool.prefix_score[:] = np.nan
    pool.completion[:] = pool.V - 1
    pool.tags[:] = pool.V - 2
    pool.completion[top] = pool.V
    for i in top:
        pool.tags[pool.offsets[i]:pool.offsets[i + 1]] = pool.V
    pool.capacity = kept
    return top


@pytest.mark.parametrize("n", [200, 256, 257, 1024, 1025, 4096, 4097, 8192])
@pytest.mark.parametrize("kind", ["short", "long"])
def test_survivors_of_other_lengths(pace, kind, n):
    pool = poolgen.make_custom_pool(_lengths(kind, n), V=40, seed=n)
    rng = np.random.default_rng(n)
    cols = [pool.tags, rng.integers(0, 256, pool.n_tokens).astype(np.uint8), rng.standard_normal(pool.n_tokens)]
    params = pace.default_params(r_max=1.0)
    for kept in (1, 4, n // 3, n):
        top = _fresh(pool, kept)
        say("ranges %s n=%d kept %d" % (kind, n, kept))
        r = oracle_step(pool, cols=cols, r_max=1.0)
        assert np.array_equal(np.flatnonzero(r["keep"]), top)
        assert_same(gpu_step(pace, pool, cols=cols, params=params, fused=True), r, "kept %d" % kept)


@pytest.mark.parametrize("n", [1000, 1025, 4096, 4097, 8192])
def test_runs_of_rejected_blocks(pace, n):
    """Kept trajectories around every 64th block, where a wave's share of the
    block sums begins, and nowhere else; then nowhere at all."""
    rng = np.random.default_rng(n)
    L = rng.integers(0, 300, n)
    off = np.concatenate([[0], np.cumsum(L)]).astype(np.int64)
    ids = rng.integers(0, 2 ** 31 - 1, int(off[-1])).astype(np.int32)
    edge = np.arange(n) // 16 % 64
    for keep in ((edge == 0), (edge == 63), (edge == 0) & (np.arange(n) % 16 == 15), np.zeros(n, bool)):
        keep = keep.astype(np.uint8)
        say("rejected blocks n=%d kept %d" % (n, keep.sum()))
        oo, kid, nk, packed = pace.pace_compact(D(off), D(keep), [D(ids)])
        torch.cuda.synchronize()
        w_off, w_ids, w = oracle.compact(off, keep, [ids])
        m = int(keep.sum())
        assert np.array_equal(H(oo)[: m + 1], w_off) and np.array_equal(H(kid)[:m], w_ids)
        assert int(H(nk)[0]) == w_off[-1] and np.array_equal(H(packed[0])[: int(w_off[-1])], w[0])


def _copy_us(pace, pool, kept):
    _fresh(pool, kept)
    d = [D(a) for a in (pool.tags, pool.offsets, pool.completion)]
    step = pace.FilterStep(pool.n, pool.n_tokens, [torch.int32], "cuda:0", pace.default_params(r_max=1.0))
    best = float("inf")
    for _ in range(20):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        b.record()
        torch.cuda.synchronize()
        pace.pace_time_next_kernel(pace.PHASE_COMPACT, a, b)
        step.run(*d, pool.V, pool.occupancy, pool.capacity, [d[0]])
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) * 1e3)
    return best


@pytest.mark.parametrize("n,short,kept,limit", [(8192, 97, 4, 40.0), (300, 20, 100, 15.0), (250, 20, 80, 22.0)])
def test_few_tokens_expected_still_fill_the_chip(pace, n, short, kept, limit):
    """4 survivors of 300,000 tokens among 8192 short ones, and survivors of 20
    tokens. With the ranges sized by the expected tokens alone the copy kernel
    takes 108, 30 and 30 us here; sized by the pool and the survivors 7, 5 and 10.
    The best of 20 runs, against limits well away from both."""
    L = np.full(n, short)
    if n == 8192:
        L[[5, 3000, 3001, 8000]] = 300000
    pool = poolgen.make_custom_pool(L, V=40, seed=1)
    us = _copy_us(pace, pool, kept)
    say("copy kernel n=%d kept %d: %.1f us" % (n, kept, us))
    assert us < limit


def _compact_us(pace, off, keep, cols):
    """The copy kernel of one pace_compact call; the best of 20 runs."""
    out = [torch.empty_like(c) for c in cols]
    best = float("inf")
    for _ in range(20):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        b.record()
        torch.cuda.synchronize()
        pace.pace_time_next_kernel(pace.PHASE_COMPACT, a, b)
        pace.pace_compact(off, keep, cols, cols_out=out)
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) * 1e3)
    return best


def test_few_tokens_over_many_blocks(pace):
    """8192 trajectories of one token, a tenth kept: a range of 16 tokens meets
    ten blocks. Block by block the copy kernel takes 15.2 us, 64 trajectories at a
    time 10.4."""
    rng = np.random.default_rng(4)
    n = 8192
    off = torch.arange(0, n + 1, dtype=torch.int64, device="cuda:0")
    us = _compact_us(pace, off, D((rng.random(n) < 0.1).astype(np.uint8)),
                     [torch.zeros(n, dtype=d, device="cuda:0") for d in (torch.int32, torch.uint8)])
    say("copy kernel, 819 of 8192 single tokens: %.1f us" % us)
    assert us < 12.8


@pytest.mark.parametrize("n", [8193, 20000])
def test_spans_of_every_length_below_a_vector(pace, n):
    """The wide copy's spans of 0 to 17 bytes, at every byte of a vector, in each
    element width (the one-byte column holds every length there is)."""
    rng = np.random.default_rng(n)
    L = rng.integers(0, 18, n)
    off = np.concatenate([[0], np.cumsum(L)]).astype(np.int64)
    keep = (rng.random(n) < 0.6).astype(np.uint8)
    N = int(off[-1])
    cols = [rng.integers(0, 256, N).astype(np.uint8), rng.integers(-9, 9, N).astype(np.int16),
            rng.integers(0, 2 ** 31 - 1, N).astype(np.int32), rng.standard_normal(N)]
    say("short spans n=%d kept %d" % (n, keep.sum()))
    oo, kid, nk, packed = pace.pace_compact(D(off), D(keep), [D(c) for c in cols])
    torch.cuda.synchronize()
    w_off, w_ids, w = oracle.compact(off, keep, cols)
    m = int(keep.sum())
    assert np.array_equal(H(oo)[: m + 1], w_off) and np.array_equal(H(kid)[:m], w_ids)
    for got, want in zip(packed, w):
        assert np.array_equal(H(got)[: int(w_off[-1])], want)


def test_spans_below_a_vector_cost_no_round_trip_a_byte(pace):
    """8 one-byte columns of 20,000 spans of 15 tokens: the copy kernel takes 26 us
    a byte at a time and 13 as it is; the best of 20 runs."""
    n = 20000
    off = torch.arange(0, n * 15 + 1, 15, dtype=torch.int64, device="cuda:0")
    keep = torch.ones(n, dtype=torch.uint8, device="cuda:0")
    cols = [torch.zeros(n * 15, dtype=torch.uint8, device="cuda:0") for _ in range(8)]
    best = _compact_us(pace, off, keep, cols)
    say("copy kernel, spans of 15 bytes: %.1f us" % best)
    assert best < 19.5

"""Scores formed by trajectory, against the oracle: lengths at the edges of a
thread's vectors, of the one, two, four and eight waves' batches and of the
tokens that one workgroup sums, trajectories summed in pieces (joined by the
rank, the group step, the streaming cutoff's launch, the separate calls' kernel
and the key extremes of larger pools), every arithmetic, and tags that start
anywhere. The pools are checked against the library's rules, so that each takes
the kernel that it names."""
import sys

import numpy as np
import pytest

import oracle
import poolgen
from tests.rules import rules
from tests.test_gpu_group import group_step_parity
from tests.test_gpu_parity import D, H, assert_same, gpu_step, oracle_step

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
CAP = 65536


def _edges(waves):
    """Lengths around a thread's four tags, the strides of 256 tokens per wave that
    a batch of eight loads takes, one batch and two, and the 16,384 (one wave),
    32,768 (two) or 65,536 tokens that a workgroup sums."""
    stride, cap = 256 * waves, min(16384 * waves, CAP)
    at = [k * stride for k in (1, 2, 4, 6, 8, 10, 16)] + [cap]
    return [0, 1, 2, 3, 4, 5, 7] + [a + d for a in at for d in (-1, 0, 1)] + [2 * cap, 2 * cap + 5]


def say(msg):
    sys.stdout.write("[gpu] %s\n" % msg)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def pace():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2609_36830_amd as pace
    return pace


def _lengths(kind):
    rng = np.random.default_rng(3)
    if kind.startswith("edges"):
        # The number of trajectories decides the waves where the mean length is small.
        waves = int(kind[5])
        L = _edges(waves) + list(rng.integers(0, 40, {8: 60, 4: 600, 2: 1100, 1: 2300}[waves]))
        n, nt = len(L), int(np.sum(L))
        assert rules().waves(n, nt) == waves and rules().cap(n, nt) == min(16384 * waves, CAP)
        return L
    if kind == "pieces8":       # several pieces, neighbours, at both ends, empty ones between
        L = [CAP + 1, 0, CAP, 2 * CAP, 2 * CAP + 1, 0, 5, CAP - 1, 3 * CAP + 777, 12, 131072, 200001]
        assert rules().waves(len(L), sum(L)) == 8
        return L
    if kind == "pieces1":       # long ones among very short ones: pieces of one wave's 16,384 tokens
        L = rng.integers(0, 30, 3000)
        L[1500], L[1501], L[2999] = CAP + 3, 150000, CAP + 1
        assert rules().waves(len(L), int(L.sum())) == 1 and rules().cap(len(L), int(L.sum())) == 16384
        return list(L)
    # "wide": above 8192 trajectories of 3072 tokens or more on average
    L = np.full(8300, 3200)
    L[rng.integers(0, 8300, 6)] = [CAP + 1, 3 * CAP, 0, 1, 100000, 65536]
    assert rules().by_traj(len(L), int(L.sum())) and rules().cap(len(L), int(L.sum())) == CAP
    return list(L)


KINDS = ["edges8", "edges4", "edges2", "edges1", "pieces8", "pieces1", "wide"]


def _pool(kind, V=300, mask=0.2, seed=1):
    pool = poolgen.make_custom_pool(_lengths(kind), V=V, seed=seed, mask_frac=mask)
    pool.capacity = max(1, pool.n // 2)
    return pool


@pytest.mark.parametrize("fused", [False, True], ids=["calls", "fused"])
@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("mode", ["effective", "raw"])
def test_step(pace, kind, mode, fused):
    pool = _pool(kind)
    say("score by trajectory %s %s fused %s tokens %d" % (kind, mode, fused, pool.n_tokens))
    assert_same(gpu_step(pace, pool, mode=mode, fused=fused), oracle_step(pool, mode=mode), kind)


@pytest.mark.parametrize("side", ["below", "at", "above"])
@pytest.mark.parametrize("kind", ["edges8", "edges4", "edges2", "edges1", "pieces8"])
def test_large_versions(pace, kind, side):
    """Both sides of the 32-bit sums' limit for every number of waves, every tag at
    the largest version."""
    L = _lengths(kind)
    n, nt = len(L), int(np.sum(L))
    most = {8: 2 ** 25 - 2}.get(rules().waves(n, nt), 2 ** 24 - 2)
    assert rules().narrow(n, nt, most) and not rules().narrow(n, nt, most + 1)
    V = {"below": most, "at": most + 1, "above": 2 ** 31 - 2}[side]
    pool = _pool(kind, V=V, seed=2)
    pool.tags[:] = np.where(pool.tags == -1, -1, V).astype(np.int32)
    pool.completion[:] = V
    say("score by trajectory %s V=%d" % (kind, V))
    assert_same(gpu_step(pace, pool, fused=True), oracle_step(pool), "%s V=%d" % (kind, V))


@pytest.mark.parametrize("kind", ["edges1", "edges2", "edges4", "edges8", "pieces8"])
def test_tags_start_anywhere(pace, kind):
    pool = _pool(kind)
    sc, S, T = oracle.score(pool.tags, pool.offsets, pool.completion, pool.V, pool.prefix_score, pool.window)
    for lead in (1, 2, 3):
        buf = torch.zeros(pool.n_tokens + lead, dtype=torch.int32, device="cuda:0")
        buf[lead:] = D(pool.tags)
        say("score by trajectory %s lead %d" % (kind, lead))
        g = pace.pace_score(buf[lead:], D(pool.offsets), D(pool.completion), pool.V, D(pool.prefix_score),
                            D(pool.window))
        assert np.array_equal(H(g[0]).view(np.int64), sc.view(np.int64))
        assert np.array_equal(H(g[1]), S) and np.array_equal(H(g[2]), T)


@pytest.mark.parametrize("W", [31, 32, 33, 4096, 4097])
def test_window_sizes(pace, W):
    """One level of the window's search and more, in one wave and in eight."""
    for kind in ("edges1", "pieces8"):
        pool = poolgen.make_custom_pool(_lengths(kind), V=90, seed=5, W=W)
        pool.prefix_score[::5] = pool.window[:: max(1, W // 7)][0]       # equal to a window entry
        say("score by trajectory %s W=%d" % (kind, W))
        assert_same(gpu_step(pace, pool, fused=True, params=pace.default_params(gamma=2)), oracle_step(pool, gamma=2),
                    "W=%d" % W)


@pytest.mark.parametrize("kind", ["pieces8", "pieces1", "wide"])
def test_group_step(pace, kind):
    pool = _pool(kind)
    rng = np.random.default_rng(8)
    for sizes in ("pairs", "ragged"):
        go = np.arange(0, pool.n + 1, 2, dtype=np.int64) if sizes == "pairs" else \
            np.sort(np.concatenate([[0], rng.integers(0, pool.n + 1, pool.n // 4), [pool.n]])).astype(np.int64)
        go[-1] = pool.n
        ng = len(go) - 1
        # Means inside the rank, except over as many groups as the larger pool's pairs.
        assert rules().in_rank(pool.n, ng) == (kind != "wide" or sizes != "pairs")
        say("group step %s %s ng=%d" % (kind, sizes, ng))
        group_step_parity(pace, pool, go, ng, max(1, ng // 2))


@pytest.mark.parametrize("kind", ["pieces8", "pieces1", "wide"])
def test_stream_step(pace, kind):
    pool = _pool(kind)
    ow, gw = oracle.StreamWindow(64), pace.StreamWindow(64, "cuda:0")
    osc, S, T = oracle.score(pool.tags, pool.offsets, pool.completion, pool.V)
    bufs, rh = None, 0.0
    for step in range(2):
        say("stream step %s %d" % (kind, step))
        bufs, rh = pace.pace_stream_step(D(pool.tags), D(pool.offsets), D(pool.completion), pool.V, pool.n,
                                         pool.capacity, [D(pool.tags)], gw, pool.n // 3,
                                         params=pace.default_params(window_min=4), r_hat_prev=rh, buffers=bufs)
        ost, okappa, odrawn, okept = oracle.stream_admit(osc, rh, ow, pool.n // 3, window_min=4)
        assert np.array_equal(H(bufs["score"])[: pool.n].view(np.int64), osc.view(np.int64))
        assert np.array_equal(H(bufs["gen_sum"])[: pool.n], S) and np.array_equal(H(bufs["gen_count"])[: pool.n], T)
        assert np.array_equal(H(bufs["status"])[: pool.n], ost) and float(H(bufs["kappa"])[0]) == okappa
        assert np.array_equal(H(gw.ring).view(np.int64), ow.ring.view(np.int64))

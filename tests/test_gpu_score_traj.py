"""Scores formed by trajectory, against the oracle: lengths at the edges of a
thread's vectors, of the two, four and eight waves' batches and of the 65,536
tokens that one workgroup sums, trajectories summed in pieces (joined by the
rank, the group step, the streaming cutoff's launch, the separate calls' kernel
and the key extremes of larger pools), every arithmetic, and tags that start
anywhere."""
import sys

import numpy as np
import pytest

import oracle
import poolgen
from tests.test_gpu_group import group_step_parity
from tests.test_gpu_parity import D, H, assert_same, gpu_step, oracle_step

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
EDGES = [0, 1, 2, 3, 4, 5, 7, 511, 512, 513, 1023, 1025, 2047, 2048, 2049, 3071, 3073, 4095, 4096, 4097, 8191, 8192,
         8193, 12287, 12289, 16383, 16384, 16385]
CAP = 65536


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
    if kind == "edges8":        # mean above 4096 tokens: eight waves
        return EDGES + [20000] * 12
    if kind == "edges4":        # four waves
        return EDGES + [600] * 60
    if kind == "edges2":        # mean below 1024: two waves
        return EDGES + list(rng.integers(0, 40, 600))
    if kind == "pieces8":       # several pieces, neighbours, at both ends, empty ones between
        return [CAP + 1, 0, CAP, 2 * CAP, 2 * CAP + 1, 0, 5, CAP - 1, 3 * CAP + 777, 12, 131072, 200001]
    if kind == "pieces2":       # long ones among very short ones
        L = list(rng.integers(0, 30, 3000))
        L[1500], L[1501], L[2999] = CAP + 3, 150000, CAP + 1
        return L
    L = np.full(8300, 2500)     # "wide": above 8192 trajectories of over 2048 tokens on average
    L[rng.integers(0, 8300, 6)] = [CAP + 1, 3 * CAP, 0, 1, 100000, 65536]
    return list(L)


KINDS = ["edges8", "edges4", "edges2", "pieces8", "pieces2", "wide"]


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


@pytest.mark.parametrize("V", [2 ** 22, 2 ** 23, 2 ** 24 - 1, 2 ** 24, 2 ** 31 - 2])
@pytest.mark.parametrize("kind", ["edges8", "edges4", "edges2", "pieces8"])
def test_large_versions(pace, kind, V):
    """Both sides of the 32-bit sums' limit for every number of waves."""
    pool = _pool(kind, V=V, seed=2)
    say("score by trajectory %s V=%d" % (kind, V))
    assert_same(gpu_step(pace, pool, fused=True), oracle_step(pool), "%s V=%d" % (kind, V))


@pytest.mark.parametrize("kind", ["edges4", "edges8", "pieces8"])
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
    """Windows counted beside the tags (up to 4096 entries) and searched."""
    for kind in ("edges2", "pieces8"):
        pool = poolgen.make_custom_pool(_lengths(kind), V=90, seed=5, W=W)
        pool.prefix_score[::5] = pool.window[:: max(1, W // 7)][0]       # equal to a window entry
        say("score by trajectory %s W=%d" % (kind, W))
        assert_same(gpu_step(pace, pool, fused=True, params=pace.default_params(gamma=2)), oracle_step(pool, gamma=2),
                    "W=%d" % W)


@pytest.mark.parametrize("kind", ["pieces8", "pieces2", "wide"])
def test_group_step(pace, kind):
    pool = _pool(kind)
    rng = np.random.default_rng(8)
    for sizes in ("pairs", "ragged"):
        go = np.arange(0, pool.n + 1, 2, dtype=np.int64) if sizes == "pairs" else \
            np.sort(np.concatenate([[0], rng.integers(0, pool.n + 1, pool.n // 4), [pool.n]])).astype(np.int64)
        go[-1] = pool.n
        ng = len(go) - 1
        say("group step %s %s ng=%d" % (kind, sizes, ng))
        group_step_parity(pace, pool, go, ng, max(1, ng // 2))


@pytest.mark.parametrize("kind", ["pieces8", "pieces2", "wide"])
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

"""Scores over equal chunks of tokens, against the oracle: pools of more than
8192 trajectories of under 3072 tokens on average, in each arithmetic of the
reduction and next to the limits between them, with tags that start anywhere and
windows beyond what the second kernel stages in LDS."""
import sys

import numpy as np
import pytest

import oracle
import poolgen
from tests.rules import NARROW, PACKED, WIDE, rules
from tests.test_gpu_parity import D, H, assert_same, gpu_step, oracle_step

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
MODES = [(32766, PACKED), (32767, NARROW), (2 ** 24 - 2, NARROW), (2 ** 24 - 1, WIDE), (2 ** 30, WIDE),
         (2 ** 31 - 2, WIDE)]


def say(msg):
    sys.stdout.write("[gpu] %s\n" % msg)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def pace():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2609_36830_amd as pace
    return pace


def _pool(kind, V, seed, mask=0.1, W=64):
    """"long": window and chunk edges and a trajectory over many chunks, then short
    ones; "short": boundaries in most windows, some trajectories empty."""
    rng = np.random.default_rng(seed)
    L = rng.integers(0, 60, 8300) if kind == "long" else np.where(rng.random(9001) < 0.2, 0, rng.integers(0, 300, 9001))
    if kind == "long":
        L[:14] = [70000, 1, 255, 256, 257, 3000, 0, 4096, 12345, 2047, 2048, 2049, 300000, 0]
        L[-2:] = [1500, 511]
    pool = poolgen.make_custom_pool(L, V=V, seed=seed, mask_frac=mask, c_lag=0, W=W)
    assert not rules().by_traj(pool.n, pool.n_tokens)
    return pool


def _largest(pool):
    """Every generated tag at V."""
    pool.tags[:] = np.where(pool.tags == -1, -1, pool.V).astype(np.int32)
    pool.completion[:] = pool.V
    return pool


@pytest.mark.parametrize("fused", [False, True], ids=["calls", "fused"])
@pytest.mark.parametrize("kind", ["long", "short"])
@pytest.mark.parametrize("V,mode", MODES)
def test_mode_limits(pace, V, mode, kind, fused):
    """Full windows of the largest tags must neither carry into the packed count
    nor overflow a 32-bit window sum."""
    pool = _largest(_pool(kind, V, V % 1000 + 1))
    assert rules().mode(V) == mode
    say("score over chunks %s V=%d fused %s" % (kind, V, fused))
    assert_same(gpu_step(pace, pool, fused=fused), oracle_step(pool), "%s V=%d" % (kind, V))


@pytest.mark.parametrize("lead", [0, 1, 2, 3])
@pytest.mark.parametrize("V", [300, 32767, 2 ** 30])
def test_tags_start_anywhere(pace, V, lead):
    """The last chunk's ragged end in every lane of the last vector too."""
    for kind in ("long", "short"):
        pool = _pool(kind, V, 5 + lead)
        sc, S, T = oracle.score(pool.tags, pool.offsets, pool.completion, pool.V, pool.prefix_score, pool.window)
        buf = torch.full((pool.n_tokens + lead,), 2 ** 31 - 1, dtype=torch.int32, device="cuda:0")
        buf[lead:] = D(pool.tags)
        say("score over chunks %s V=%d lead %d tokens %d" % (kind, V, lead, pool.n_tokens))
        g = pace.pace_score(buf[lead:], D(pool.offsets), D(pool.completion), pool.V, D(pool.prefix_score),
                            D(pool.window))
        assert np.array_equal(H(g[0]).view(np.int64), sc.view(np.int64))
        assert np.array_equal(H(g[1]), S) and np.array_equal(H(g[2]), T)


@pytest.mark.parametrize("fused", [False, True], ids=["calls", "fused"])
@pytest.mark.parametrize("W", [31, 32, 4096, 4097, 6000])
def test_window_sizes(pace, W, fused):
    """Windows staged in LDS (up to 4096 entries) and searched in global memory."""
    pool = _pool("short", 90, W, W=W)
    pool.prefix_score[::5] = pool.window[:: max(1, W // 7)][0]       # equal to a window entry
    say("score over chunks W=%d fused %s" % (W, fused))
    assert_same(gpu_step(pace, pool, fused=fused, params=pace.default_params(gamma=1)), oracle_step(pool, gamma=1),
                "W=%d" % W)

"""The prefix window's count in the scores by trajectory: sizes at the edges of
the 64-way search's levels, prefix scores equal to entries, between, below and
above them, repeated entries, and that a large window costs no more than a small
one, by the score kernel's own time."""
import sys

import numpy as np
import pytest

import oracle
import poolgen
from tests.test_gpu_parity import D, H

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


@pytest.mark.parametrize("W", [1, 2, 31, 63, 64, 65, 127, 128, 129, 512, 4032, 4095, 4096, 4097, 6000, 64 * 64 * 64 + 1])
@pytest.mark.parametrize("n", [90, 2600])
def test_counts(pace, n, W):
    """90 trajectories take eight waves each, 2600 one."""
    rng = np.random.default_rng(W + n)
    pool = poolgen.make_custom_pool(rng.integers(0, 60, n), V=50, seed=W % 97 + n)
    win = np.sort(np.where(rng.random(W) < 0.3, 0.5, rng.random(W)))        # a run of equal entries
    at = rng.integers(0, W, n)
    pre = np.where(rng.random(n) < 0.5, win[at], np.nextafter(win[at], rng.choice([-1.0, 2.0], n)))
    pre[:12] = [np.nan, np.inf, -np.inf, win[0], win[-1], np.nextafter(win[0], -1), np.nextafter(win[-1], 2), 0.5,
                0.0, -0.0, 0.25, 0.75]
    params = pace.default_params(gamma=1, window_min=1)
    sc, S, T = oracle.score(pool.tags, pool.offsets, pool.completion, pool.V, pre, win, gamma=1, window_min=1)
    say("window of %d, %d trajectories" % (W, n))
    g = pace.pace_score(D(pool.tags), D(pool.offsets), D(pool.completion), pool.V, D(pre), D(win), params)
    assert np.array_equal(H(g[0]).view(np.int64), sc.view(np.int64))
    assert np.array_equal(H(g[1]), S) and np.array_equal(H(g[2]), T)


def test_large_window_costs_no_more(pace):
    """8192 trajectories of 500 tokens: with every entry loaded by every
    workgroup the kernel takes 7 us with 64 entries and 22 with 4096. The best
    of 20 runs each."""
    n, N = 8192, 8192 * 500
    off = torch.arange(0, N + 1, 500, dtype=torch.int64, device="cuda:0")
    tags = torch.full((N,), 3, dtype=torch.int32, device="cuda:0")
    comp = torch.full((n,), 5, dtype=torch.int32, device="cuda:0")
    pre = torch.rand(n, dtype=torch.float64, device="cuda:0")
    us = {}
    for W in (64, 4096):
        win = torch.sort(torch.rand(W, dtype=torch.float64, device="cuda:0"))[0]
        us[W] = float("inf")
        for _ in range(20):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            b.record()
            torch.cuda.synchronize()
            pace.pace_time_next_kernel(pace.PHASE_REDUCE, a, b)
            pace.pace_score(tags, off, comp, 7, pre, win)
            torch.cuda.synchronize()
            us[W] = min(us[W], a.elapsed_time(b) * 1e3)
    say("score kernel: %.1f us with 64 entries, %.1f with 4096" % (us[64], us[4096]))
    assert us[4096] < 1.5 * us[64]

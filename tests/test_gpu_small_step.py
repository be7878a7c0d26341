"""Filter steps whose selection and compaction are one kernel (small pools), and
their neighbours on the other side of its limits, against the oracle: partial
waves, ties, every budget edge, empty trajectories, several columns, and
trajectories summed in pieces."""
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


def _check(pace, pool, what, cols=None, **kw):
    say(what)
    r = oracle_step(pool, cols=cols, **{k: v for k, v in kw.items() if k != "params"})
    assert_same(gpu_step(pace, pool, cols=cols, fused=True, params=kw.get("params")), r, what)


@pytest.mark.parametrize("n", [0, 1, 2, 63, 64, 65, 127, 128, 129, 191, 255, 256, 257])
def test_sizes_and_budgets(pace, n):
    rng = np.random.default_rng(n)
    L = rng.integers(0, 700, n)
    L[rng.random(n) < 0.15] = 0
    for cap in sorted({0, 1, n // 2, max(0, n - 1), n, n + 3}):
        pool = poolgen.make_custom_pool(L, V=40, seed=n, mask_frac=0.2, capacity=cap)
        _check(pace, pool, "small n=%d capacity=%d" % (n, cap), r_max=1.0, params=pace.default_params(r_max=1.0))


@pytest.mark.parametrize("n", [40, 200])
def test_ties(pace, n):
    """Equal scores across waves: the lower ids go first."""
    pool = poolgen.make_custom_pool(np.full(n, 30), V=9, seed=3, max_breaks=0, c_lag=2)
    pool.prefix_score[:] = np.nan
    for cap in (1, n // 3, n // 2, n - 2):
        pool.capacity = cap
        _check(pace, pool, "small ties n=%d capacity=%d" % (n, cap))


@pytest.mark.parametrize("n,mean", [(100, 7000), (128, 16000), (128, 17500), (129, 8000), (256, 4000), (256, 4200)])
def test_both_sides_of_the_copy_limit(pace, n, mean):
    rng = np.random.default_rng(mean)
    L = rng.integers(mean // 2, mean * 3 // 2, n)
    L[n // 2] = 70000
    pool = poolgen.make_custom_pool(L, V=40, seed=n, capacity=n // 2)
    N = pool.n_tokens
    one = [rng.integers(0, 256, N).astype(np.uint8)]
    _check(pace, pool, "small n=%d tokens=%d one column" % (n, N), cols=one)
    three = [pool.tags, (np.arange(N) % 30000).astype(np.int16), rng.standard_normal(N)]
    _check(pace, pool, "small n=%d tokens=%d three columns" % (n, N), cols=three)


def test_no_columns_and_repeats(pace):
    """Without columns, and twice on the same outputs: nothing carries over."""
    pool = poolgen.make_custom_pool(np.arange(150) * 5, V=40, seed=4, capacity=60)
    r = oracle_step(pool, cols=[])
    for _ in range(2):
        assert_same(gpu_step(pace, pool, cols=[], fused=True), r, "no columns")

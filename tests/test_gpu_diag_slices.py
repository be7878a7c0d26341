"""pace_diagnostics around the limit of its one-launch form and beyond one
round of the slices' workgroups (131,072 trajectories), against the oracle;
outputs are overwritten, not added to."""
import numpy as np
import pytest

import oracle
from tests.test_gpu_diag import D, H, _direct_pool, say

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pace():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2609_36830_amd as pace
    return pace


@pytest.mark.parametrize("n,nb", [(6144, 257), (6145, 257), (6145, 1024), (12288, 256), (12289, 1), (12289, 256),
                                  (12289, 65), (14336, 64), (14337, 33), (14337, 64), (16384, 32), (16385, 1), (16385, 32),
                                  (65536, 64), (131072 + 1025, 63)])
def test_diagnostics_slices(pace, n, nb):
    rng = np.random.default_rng(n + nb)
    V = 40
    tags, off, comp = _direct_pool(rng, n, V)
    score, S, T = oracle.score(tags, off, comp, V)
    pick = rng.integers(0, n, n // 7)
    score[pick] = rng.choice([np.nan, np.inf, -np.inf, 0.0, 3.0, 12.0], pick.size)
    keep = rng.choice(np.array([0, 1, 2, 255], np.uint8), n)
    edges = np.sort(rng.integers(-1, 13, (3, nb + 1)), axis=1).astype(np.float64)   # repeated, hit exactly
    edges[2] = np.sort(rng.uniform(-1, 30, nb + 1))
    oh, ot = oracle.diagnostics(tags, off, comp, V, score, keep, edges)
    hist = torch.full((3, 2, nb + 2), -7, dtype=torch.int64, device="cuda:0")
    totals = torch.full((2, 4), -7, dtype=torch.int64, device="cuda:0")
    for _ in range(2):
        say("diagnostics slices n=%d nbins=%d" % (n, nb))
        pace.pace_diagnostics(D(score), D(S), D(T), D(comp), V, D(keep), D(edges), hist, totals)
        assert np.array_equal(H(hist), oh) and np.array_equal(H(totals), ot)

"""pace_compact on columns of every width at every byte alignment, against the
oracle: spans around the 16-byte vectors and the wave/workgroup split of the
copy, ranges that skip long runs of rejected trajectories, and nothing written
past the packed batch."""
import sys

import numpy as np
import pytest

import oracle
from tests.test_gpu_parity import D, H

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
SENTINEL = 0x5A


@pytest.fixture(scope="module")
def pace():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2609_36830_amd as pace
    return pace


def _lengths(kind, rng):
    if kind == "short":       # around one vector of every width
        return rng.integers(0, 40, 700)
    if kind == "split":       # around kWaveCopy bytes of every width, and range ends inside spans
        return np.concatenate([rng.integers(240, 2100, 300), [2047, 2048, 2049, 511, 512, 513, 255, 256, 257]])
    if kind == "long":        # spans over many ranges
        return np.array([3, 70001, 0, 16, 40000, 1, 15, 120007])
    return rng.integers(0, 60, 9000)     # wide: blocks of 64


@pytest.mark.parametrize("kind", ["short", "split", "long", "wide"])
@pytest.mark.parametrize("pattern", ["random", "ends"])
def test_compact_alignments(pace, kind, pattern):
    rng = np.random.default_rng(len(kind) + 7 * len(pattern))
    L = _lengths(kind, rng)
    n = len(L)
    off = np.concatenate([[0], np.cumsum(L)]).astype(np.int64)
    N = int(off[-1])
    keep = (rng.random(n) < 0.5).astype(np.uint8)
    if pattern == "ends":                # kept trajectories only at the two ends
        keep[:] = 0
        keep[: 1 + n // 50] = 1
        keep[-1 - n // 50:] = 1
    for shift in range(0, 16, 1 if kind in ("short", "wide") else 3):
        # Two columns of each width, the outputs at another alignment than the inputs.
        host, cin, bufs, cout = [], [], [], []
        for k, dt in enumerate((np.uint8, np.int16, np.int32, np.float64)):
            e = np.dtype(dt).itemsize
            raw = rng.integers(0, 256, N * e, dtype=np.uint8)
            a, b = shift // e * e, (shift * 5 + k) % 16 // e * e
            dev = torch.zeros(N * e + 32, dtype=torch.uint8, device="cuda:0")
            dev[a:a + N * e] = D(raw)
            out = torch.full((N * e + 64,), SENTINEL, dtype=torch.uint8, device="cuda:0")
            host.append(raw.view(dt))
            tdt = torch.from_numpy(np.zeros(1, dt)).dtype
            cin.append(dev[a:a + N * e].view(tdt) if a % e == 0 else None)
            bufs.append((out, b))
            cout.append(out[b:b + N * e].view(tdt))
        sys.stdout.write("[gpu] compact %s %s shift %d\n" % (kind, pattern, shift))
        sys.stdout.flush()
        oo, ids, nk, _ = pace.pace_compact(D(off), D(keep), cin, cols_out=cout, n_tokens=N)
        torch.cuda.synchronize()
        want_off, want_ids, want = oracle.compact(off, keep, host)
        m = int(keep.sum())
        assert np.array_equal(H(oo)[: m + 1], want_off) and np.array_equal(H(ids)[:m], want_ids)
        assert int(H(nk)[0]) == int(want_off[-1])
        for (out, b), w in zip(bufs, want):
            got = H(out)
            nb = w.nbytes
            assert np.array_equal(got[b:b + nb], w.view(np.uint8)), (kind, shift, w.dtype)
            assert (got[:b] == SENTINEL).all() and (got[b + nb:] == SENTINEL).all(), "written outside the batch"

"""pace_validate's tag check at the edges of its chunks (8192 tokens), vectors
and trajectories: a version one above its trajectory's completion, planted at
each edge, is found; one equal to it is not. Malformed offsets give the flags of
the documented walk."""
import sys

import numpy as np
import pytest

import oracle
from tests.test_gpu_parity import D, H

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
V = 100


@pytest.fixture(scope="module")
def pace():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2609_36830_amd as pace
    return pace


def _pool(kind, rng):
    if kind == "mixed":
        L = np.concatenate([[0, 1, 2, 3, 4, 5, 0, 0], rng.integers(0, 9, 150), [1023, 1025, 8190, 2, 8192, 1],
                            np.zeros(200, np.int64), rng.integers(200, 3000, 12), [0, 0, 7]])
    elif kind == "long":
        L = np.array([30001, 1, 50000])
    else:
        L = rng.integers(0, 3, 9000)
    off = np.concatenate([[0], np.cumsum(L)]).astype(np.int64)
    comp = rng.integers(0, V + 1, len(L)).astype(np.int32)
    tags = np.repeat(comp, L).astype(np.int32)           # every tag equals its completion version
    tags[rng.random(len(tags)) < 0.2] = -1
    return off, comp, tags


def _run(pace, tags, off, comp, lead=0):
    buf = torch.zeros(len(tags) + lead, dtype=torch.int32, device="cuda:0")
    buf[lead:] = D(tags)
    e = pace.pace_validate(buf[lead:], D(off), D(comp), V)
    torch.cuda.synchronize()
    return int(H(e)[0])


@pytest.mark.parametrize("kind", ["mixed", "long", "tiny"])
def test_bad_tag_at_every_edge(pace, kind):
    rng = np.random.default_rng(5)
    off, comp, tags = _pool(kind, rng)
    N, n = len(tags), len(comp)
    traj = np.repeat(np.arange(n), np.diff(off))
    assert oracle.validate(tags, off, comp, V) == 0
    at = {0, 1, 2, 3, 4, N - 1, N - 2, N - 4, N - 5}
    at |= {p + d for p in range(8192, N, 8192) for d in (-5, -4, -1, 0, 1, 3)}
    at |= {int(p) + d for p in rng.choice(off, 12) for d in (-1, 0, 1)}
    at |= {p + d for p in (256, 1024, 2048, 3072) for d in (-1, 0)}
    at = sorted(p for p in at if 0 <= p < N)
    for lead in (0, 1, 3):
        sys.stdout.write("[gpu] validate %s lead %d tokens %d\n" % (kind, lead, N))
        sys.stdout.flush()
        assert _run(pace, tags, off, comp, lead) == 0
        for p in at:
            for bad in (int(comp[traj[p]]) + 1, -2):
                t = tags.copy()
                t[p] = bad
                assert oracle.validate(t, off, comp, V) != 0
                assert _run(pace, t, off, comp, lead) == pace.BAD_TAG, (p, bad)


def _walk(tags, off, comp, chunk=8192):
    """The tag flag by the walk that the kernel documents, token by token."""
    n, N = len(comp), len(tags)
    for cs in range(0, N, chunk):
        ce = min(cs + chunk, N)
        a, base, ln = off, 0, n + 1                      # the kernel's 64-ary search for the last offset <= cs
        cur = None
        while ln > 64:
            step = (ln + 63) // 64
            cnt = sum(1 for k in range(64) if base + k * step < base + ln and a[base + k * step] <= cs)
            if cnt == 0:
                cur = base - 1
                break
            nb = base + (cnt - 1) * step
            ln = min(base + ln - nb, step)
            base = nb
        if cur is None:
            cur = base + sum(1 for k in range(ln) if a[base + k] <= cs) - 1
        cur = max(cur, 0)
        clip = lambda x: min(max(int(x), 0), N)
        while cur < n and clip(off[cur + 1]) <= cs:
            cur += 1
        for w in range(cs, ce, 64):
            lo, we = w, min(w + 64, ce)
            while cur < n:
                hi = clip(off[cur + 1])
                x = tags[lo if lo > w else w:min(hi, we)]
                if ((x != -1) & ((x < 0) | (x > comp[cur]))).any():
                    return True
                if hi >= we:
                    break
                lo = hi
                cur += 1
    return False


def test_malformed_offsets_give_the_walks_flags(pace):
    rng = np.random.default_rng(11)
    for k in range(24):
        off, comp, tags = _pool("mixed" if k % 2 else "tiny", rng)
        bad = off.copy()
        j = rng.integers(0, len(off), 1 + k % 5)
        bad[j] = rng.integers(-5, len(tags) + 5, len(j))
        want = pace.BAD_TAG if _walk(tags, bad, comp) else 0
        mono = (np.diff(bad) >= 0).all() and bad[0] == 0 and bad[-1] == len(tags)
        want |= 0 if mono else pace.BAD_OFFSETS
        sys.stdout.write("[gpu] validate malformed %d want %d\n" % (k, want))
        sys.stdout.flush()
        assert _run(pace, tags, bad, comp) == want


def _short(kind, rng):
    """Trajectories that a wave takes one per lane, and their neighbours: over 128
    tokens on average, a lane's share of 16 tokens per trajectory of the batch
    and one more (64 and 9 of them), batches cut by a chunk's end, by the last
    trajectory and by empty ones, and fewer than four tokens in all."""
    L = {"mean": rng.integers(100, 157, 400), "most": np.r_[rng.integers(0, 40, 70), 1024, rng.integers(0, 40, 90), 1025,
                                                          rng.integers(0, 40, 333)],
         "share": np.r_[np.full(63, 3), 1024, np.full(63, 3), 1025, np.full(63, 3), 1009, np.full(8, 3), 144],
         "share9": np.r_[np.full(4, 3), 145, np.full(4, 3)],
         "empty": np.where(rng.random(2000) < 0.9, 0, rng.integers(1, 300, 2000)),
         "steps": np.tile([15, 16, 17, 1, 31, 32, 33, 0], 90), "few": np.array([1, 0, 2]), "four": np.array([0, 1, 3])}[kind]
    off = np.concatenate([[0], np.cumsum(L)]).astype(np.int64)
    comp = rng.integers(0, V + 1, len(L)).astype(np.int32)
    tags = np.repeat(comp, L).astype(np.int32)
    tags[rng.random(len(tags)) < 0.2] = -1
    return off, comp, tags


@pytest.mark.parametrize("kind", ["mean", "most", "share", "share9", "empty", "steps", "few", "four"])
def test_bad_tag_in_short_trajectories(pace, kind):
    rng = np.random.default_rng(7)
    off, comp, tags = _short(kind, rng)
    N, n = len(tags), len(comp)
    traj = np.repeat(np.arange(n), np.diff(off))
    at = {0, 1, 2, N - 1, N - 2, N - 3, N - 4, N - 5} | {p + d for p in range(8192, N, 8192) for d in (-2, -1, 0, 1)}
    at |= {int(p) + d for p in rng.choice(off, 40) for d in (-2, -1, 0, 1)}
    for lead in (0, 1):
        sys.stdout.write("[gpu] validate short %s lead %d tokens %d\n" % (kind, lead, N))
        sys.stdout.flush()
        assert _run(pace, tags, off, comp, lead) == 0
        for p in sorted(p for p in at if 0 <= p < N):
            for bad in (int(comp[traj[p]]) + 1, -2):
                t = tags.copy()
                t[p] = bad
                assert _run(pace, t, off, comp, lead) == pace.BAD_TAG, (p, bad)


@pytest.mark.parametrize("kind", ["mean", "most", "share", "empty", "steps"])
def test_malformed_short_trajectories_give_the_walks_flags(pace, kind):
    rng = np.random.default_rng(13)
    off, comp, tags = _short(kind, rng)
    for k in range(12):
        bad = off.copy()
        j = rng.integers(0, len(off), 1 + k % 4)
        bad[j] = bad[j] + rng.integers(-300, 300, len(j)) if k % 2 else rng.integers(-5, len(tags) + 5, len(j))
        want = pace.BAD_TAG if _walk(tags, bad, comp) else 0
        mono = (np.diff(bad) >= 0).all() and bad[0] == 0 and bad[-1] == len(tags)
        want |= 0 if mono else pace.BAD_OFFSETS
        sys.stdout.write("[gpu] validate malformed short %s %d want %d\n" % (kind, k, want))
        sys.stdout.flush()
        assert _run(pace, tags, bad, comp) == want


def _call_us(pace, lengths):
    """A call on trajectories of these lengths: calls back to back, the best of
    five rounds."""
    off = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    tags = torch.full((int(off[-1]),), 3, dtype=torch.int32, device="cuda:0")
    comp = torch.full((len(lengths),), 5, dtype=torch.int32, device="cuda:0")
    off = D(off)
    err = torch.zeros(1, dtype=torch.int32, device="cuda:0")
    us = []
    for _ in range(5):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        pace.pace_validate(tags, off, comp, V, err_out=err)
        a.record()
        for _ in range(20):
            pace.pace_validate(tags, off, comp, V, err_out=err)
        b.record()
        torch.cuda.synchronize()
        us.append(a.elapsed_time(b) * 1e3 / 20)
    assert int(H(err)[0]) == 0
    return min(us)


def test_short_trajectories_do_not_cost_a_round_trip_each(pace):
    """200,000 trajectories of 20 tokens: 245 us a call with the trajectories of
    a chunk one after the other, 18 with one per lane."""
    us = _call_us(pace, np.full(200000, 20))
    sys.stdout.write("[gpu] validate 200,000 trajectories of 20 tokens: %.1f us\n" % us)
    assert us < 120


def test_a_long_among_few_short_trajectories(pace):
    """15 trajectories of 5 tokens and one of 1000 against 16 of as many tokens
    together: 25 us a call with one per lane wherever none is above 1024 tokens (a
    lane with 1000 takes 63 round trips), 9.4 as it is; the even ones 6.8. The limit
    lies between the two ratios, and calls that a slow host spaces further apart only
    lower them."""
    us, even = _call_us(pace, np.r_[np.full(8, 5), 1000, np.full(7, 5)]), _call_us(pace, np.full(16, 67))
    sys.stdout.write("[gpu] validate one long: %.1f us, even %.1f\n" % (us, even))
    assert us < 2.2 * even


def test_lanes_without_tokens_left_do_not_read_on(pace):
    """262,144 log-normal lengths of 100 on average: 201 us a call with one per
    lane and every lane reading as long as the longest, 85 as it is, 84 one after
    the other."""
    w = np.exp(np.random.default_rng(1).standard_normal(262144))
    us = _call_us(pace, (w / w.sum() * len(w) * 100).astype(np.int64))
    sys.stdout.write("[gpu] validate log-normal: %.1f us\n" % us)
    assert us < 140

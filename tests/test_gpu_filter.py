"""The filtered sweep (large graphs whose heads are scattered) against the
round-by-round path, which gathers every value: at its smallest sizes, with
rows beyond a wave's and a workgroup's share, ties, edge times, values spread
over more than the codes' range, and heads that switch it off."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1111_0627_amd import ocm, synth

pytestmark = pytest.mark.gpu

N = 3 << 19


def both(rp, col, w, mode="min", t=None):
    dev = [torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in (rp, col, w)]
    kw = dict(want_policy=True, want_potential=True)
    if t is None:
        def fn(**k):
            return ocm.cycle_mean(*dev, mode=mode, **kw, **k)
    else:
        tt = torch.from_numpy(t).cuda()

        def fn(**k):
            f = ocm.min_cycle_ratio if mode == "min" else ocm.max_cycle_ratio
            return f(*dev, tt, **kw, **k)
    a, b = fn(), fn(schedule=8)
    same = ("p", "q", "W", "L", "source", "iterations", "flags", "tight_edges", "fast_iters",
            "connect_rounds")
    assert [getattr(a, k) for k in same] == [getattr(b, k) for k in same]
    for k in ("cycle_edges", "policy", "potential"):
        assert torch.equal(getattr(a, k), getattr(b, k)), k


def graph(n, weights, seed, long_rows=()):
    """A ring, random further edges, and a few rows of the given degrees."""
    r = np.random.default_rng(seed)
    deg = r.integers(1, 6, n)
    for i, d in enumerate(long_rows):
        deg[(i * n) // max(len(long_rows), 1) + 3] = d
    rp = np.zeros(n + 1, np.int32)
    rp[1:] = np.cumsum(deg)
    col = r.integers(0, n, rp[-1]).astype(np.int32)
    col[rp[:-1]] = (np.arange(n) + 1) % n
    lo, hi, dt = weights
    return rp, col, r.integers(lo, hi, rp[-1]).astype(dt)


@pytest.mark.parametrize("n,weights,long_rows", [
    (N - 1, (-1000, 1000, np.int64), ()),
    (N, (-1000, 1000, np.int32), ()),
    (N + 1, (0, 2, np.int32), ()),                        # ties
    (N + 77, (-100, 100, np.int64), (31, 32, 33, 64, 1535, 1536, 1537, 4000)),
    (N + 256, (-20000, 20000, np.int64), (70000, 8193, 33)),   # giant rows; values near int32's end
    (N, (5, 6, np.int64), ()),                            # one weight: every value zero
])
def test_graphs(n, weights, long_rows):
    both(*graph(n, weights, [81, n], long_rows), mode="min" if n % 2 else "max")


@pytest.mark.parametrize("dt", [np.int32, np.int64])
def test_times(dt):
    rp, col, w = graph(N + 5, (-300, 300, dt), 82, (40, 3000))
    t = np.random.default_rng(3).integers(1, 9, len(w)).astype(np.int32)
    both(rp, col, w, "min", t)


@pytest.mark.parametrize("near", [8, 512, 8192])
def test_heads_near_their_tail(near):
    """Lines shared by many heads: the values are gathered as before."""
    rp, col, w = graph(N, (-50, 50, np.int64), 83)
    tail = np.repeat(np.arange(N), np.diff(rp))
    off = np.random.default_rng(near).integers(0, near, len(col))
    off[rp[:-1]] = 1
    both(rp, ((tail + off) % N).astype(np.int32), w)


def test_warm_start():
    rp, col, w = graph(N + 3, (-1000, 1000, np.int64), 84)
    dev = [torch.from_numpy(x).cuda() for x in (rp, col, w)]
    a = ocm.cycle_mean(*dev, want_policy=True)
    w2 = torch.from_numpy(w + np.random.default_rng(1).integers(-9, 9, len(w))).cuda()
    x = ocm.cycle_mean(dev[0], dev[1], w2, init_policy=a.policy, want_policy=True, want_potential=True)
    y = ocm.cycle_mean(dev[0], dev[1], w2, init_policy=a.policy, want_policy=True, want_potential=True,
                       schedule=8)
    assert (x.p, x.q, x.iterations, x.tight_edges) == (y.p, y.q, y.iterations, y.tight_edges)
    assert torch.equal(x.potential, y.potential) and torch.equal(x.policy, y.policy)


@pytest.mark.parametrize("n,long_rows", [(N, ()), (N + 1, (9, 8192, 7000, 33)), ((1 << 21) + 5, (8191,))])
def test_reverse_csr_of_scattered_heads(n, long_rows):
    """Push rounds (which read the reverse CSR) against pull rounds."""
    dev = [torch.from_numpy(x).cuda() for x in graph(n, (-1000, 1000, np.int32), [85, n], long_rows)]
    a, b = (ocm.cycle_mean(*dev, connect=k, want_policy=True, want_potential=True) for k in ("auto", "pull"))
    assert (a.p, a.q, a.iterations, a.connect_rounds) == (b.p, b.q, b.iterations, b.connect_rounds)
    assert torch.equal(a.policy, b.policy) and torch.equal(a.potential, b.potential)

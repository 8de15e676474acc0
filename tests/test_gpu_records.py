"""The cycle step by records against the round-by-round path, on policies whose
cycles have the lengths where it changes its form (a thread's walk, a
workgroup's queue, beyond it), many or few of them, paths in order of the
vertices and against it, and paths that take too many steps."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1111_0627_amd import ocm

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def large_path(monkeypatch):
    monkeypatch.setenv("OCM_SMALL", "0")


def both(f, weights, mode="min", t=None, seed=0):
    """Vertex v's light edge goes to f[v], a heavy one to v + 1: the first
    policy is f, and the graph is strongly connected."""
    n = len(f)
    r = np.random.default_rng(seed)
    rp = np.arange(0, 2 * n + 1, 2, dtype=np.int32)
    col = np.empty(2 * n, np.int32)
    w = np.empty(2 * n, weights)
    swap = r.integers(0, 2, n)
    at = np.arange(n) * 2
    col[at + swap], w[at + swap] = f, r.integers(-40, 40, n)
    col[at + 1 - swap], w[at + 1 - swap] = (np.arange(n) + 1) % n, r.integers(60, 900, n)
    if mode == "max":
        w = -w
    dev = [torch.from_numpy(x).cuda() for x in (rp, col, w)]
    kw = dict(want_policy=True, want_potential=True)
    if t is None:
        def fn(**k):
            return ocm.cycle_mean(*dev, mode=mode, **kw, **k)
    else:
        tt = torch.from_numpy(r.integers(1, t, 2 * n).astype(np.int32)).cuda()

        def fn(**k):
            g = ocm.min_cycle_ratio if mode == "min" else ocm.max_cycle_ratio
            return g(*dev, tt, **kw, **k)
    a, b = fn(), fn(schedule=8)
    same = ("p", "q", "W", "L", "source", "iterations", "flags", "tight_edges", "fast_iters",
            "connect_rounds")
    assert [getattr(a, k) for k in same] == [getattr(b, k) for k in same]
    for k in ("cycle_edges", "policy", "potential"):
        assert torch.equal(getattr(a, k), getattr(b, k)), k


def cycles(n, length, shuffle, tails=0):
    """Cycles of the given length over all vertices but the last `tails`,
    which lead into them in a path."""
    r = np.random.default_rng(length)
    order = r.permutation(n) if shuffle else np.arange(n)
    k = (n - tails) // length * length
    f = np.empty(n, np.int32)
    body = order[:k].reshape(-1, length)
    f[body] = np.roll(body, -1, 1)
    rest = order[k:]
    f[rest] = np.concatenate([order[:1], rest[:-1]]) if len(rest) else rest
    return f


@pytest.mark.parametrize("length", [1, 2, 47, 48, 49, 255, 256, 257, 3000])
@pytest.mark.parametrize("shuffle", [False, True])
def test_lengths(length, shuffle):
    both(cycles(20011, length, shuffle, tails=500), np.int64 if shuffle else np.int32,
         "max" if length % 2 else "min", seed=length)


@pytest.mark.parametrize("length", [8191, 8192, 8193, 30000])
def test_a_workgroups_queue(length):
    both(cycles(30011, length, True), np.int32, seed=length)


def test_times():
    both(cycles(10007, 100, True, tails=300), np.int64, "max", t=9, seed=3)
    both(cycles(10007, 7, True, tails=300), np.int32, "min", t=9, seed=4)


@pytest.mark.parametrize("n", [1, 2, 255, 257, (1 << 18) - 1, (1 << 18) + 1])
def test_random_heads(n):
    both(np.random.default_rng(n).integers(0, n, n).astype(np.int32), np.int64, seed=n)


@pytest.mark.parametrize("step", [1, -1])
def test_paths_in_order(step):
    n = 50000
    f = (np.arange(n) + step).clip(0, n - 1).astype(np.int32)
    both(f, np.int32, seed=1)


@pytest.mark.parametrize("down", [True, False])
def test_paths_in_the_order_of_the_records(down):
    """Every vertex a record of the one before, or none of them for long."""
    n = 6000
    key = (np.arange(n, dtype=np.uint64) * 0x9E3779B1 % (1 << 32)).astype(np.int64)
    order = np.argsort(-key if down else key)
    f = np.empty(n, np.int32)
    f[order[:-1]] = order[1:]
    f[order[-1]] = order[-1]
    both(f, np.int64, seed=2)


def test_batched(monkeypatch):
    """One batch of such policies against the jump rounds (kept by sweeps with
    lanes per vertex); two graphs' cycles are too long for the records."""
    monkeypatch.setenv("OCM_BATCH_SMALL", "0")
    monkeypatch.setenv("OCM_BATCH_SOLO", "0")
    r = np.random.default_rng(5)
    fs = [cycles(4000, length, True, tails=700) for length in (1, 2, 47, 48, 49, 257, 3000)]
    fs += [cycles(9000, 8192, True), cycles(9000, 8193, True), cycles(20000, 20000, True)]
    fs += [r.integers(0, n, n).astype(np.int32) for n in (1, 2, 255, 257, 5000, 60000)]
    fs += [(np.arange(5000) + d).clip(0, 4999).astype(np.int32) for d in (1, -1)]
    ns = [len(f) for f in fs]
    vptr = np.concatenate([[0], np.cumsum(ns)])
    col = np.empty(2 * vptr[-1], np.int32)
    w = np.empty(2 * vptr[-1], np.int32)
    for f, v0 in zip(fs, vptr):
        at = 2 * (v0 + np.arange(len(f)))
        col[at], w[at] = v0 + f, r.integers(-40, 40, len(f))
        col[at + 1], w[at + 1] = v0 + (np.arange(len(f)) + 1) % len(f), r.integers(60, 900, len(f))
    rp = np.arange(0, 2 * vptr[-1] + 1, 2, dtype=np.int32)
    dev = [torch.from_numpy(x).cuda() for x in (rp, col, w)]
    got = []
    for kw in (dict(), dict(schedule=8)):
        x = ocm.cycle_mean_batched(*dev, vptr, 2 * vptr, **kw)
        assert x.status == [0] * len(fs)
        got.append((x.p, x.q, x.iterations, x.flags, x.cycle_ptr, x.cycle_edges.cpu().tolist()))
    assert got[0] == got[1]


def batch_of(fs, weight):
    """The graphs of both(), as one batch; weight(g) gives graph g's light edges."""
    vptr = np.concatenate([[0], np.cumsum([len(f) for f in fs])])
    col = np.empty(2 * vptr[-1], np.int32)
    w = np.empty(2 * vptr[-1], np.int32)
    for g, (f, v0) in enumerate(zip(fs, vptr)):
        at = 2 * (v0 + np.arange(len(f)))
        col[at], w[at] = v0 + f, weight(g)
        col[at + 1], w[at + 1] = v0 + (np.arange(len(f)) + 1) % len(f), 900
    rp = np.arange(0, 2 * vptr[-1] + 1, 2, dtype=np.int32)
    return [torch.from_numpy(x).cuda() for x in (rp, col, w)], vptr


@pytest.mark.parametrize("fill", [0x00, 0xA5, 0x5A])
def test_batched_long_cycles_among_others(fill, monkeypatch):
    """Graphs left to the jump rounds whose long cycle competes with others, of
    better and worse mean at lower and higher indices, and so many of them that
    the heads of two passes together would be more than the vertices; whatever
    the workspace holds before."""
    monkeypatch.setenv("OCM_BATCH_SMALL", "0")
    r = np.random.default_rng(11)
    fs = []
    for g in range(6):
        n, long = 24000, 8193 + 97 * g
        lo = (3000, 0, 11000, 5, 6000, 11001)[g]       # where the long cycle begins
        body = lo + r.permutation(long)                # its successors shuffled
        f = np.empty(n, np.int32)
        f[body] = np.roll(body, -1)
        rest = np.setdiff1d(np.arange(n), body)
        f[rest] = rest
        if g == 0:                                     # cycles of seven, else self-loops
            k = len(rest) // 7 * 7
            f[rest[:k]] = np.roll(rest[:k].reshape(-1, 7), -1, 1).ravel()
        fs.append(f)
    fs.append(np.arange(40000, dtype=np.int32))        # nothing but self-loops

    def weight(g):
        x = r.integers(10, 500, len(fs[g]))
        if g in (0, 3, 5):   # the long cycle wins
            x[np.arange(len(x)) == fs[g]] = 500
            x[fs[g] != np.arange(len(x))] //= 2
        return x

    dev, vptr = batch_of(fs, weight)
    got = []
    for kw in (dict(), dict(schedule=8)):
        ocm.release_workspace()
        ocm.cycle_mean_batched(*dev, vptr, 2 * vptr, max_iters=1)   # makes the workspace
        for ws in ocm._bws_cache.values():
            ws.fill_(fill)
        x = ocm.cycle_mean_batched(*dev, vptr, 2 * vptr, **kw)
        assert x.status == [0] * len(fs)
        got.append((x.p, x.q, x.iterations, x.flags, x.cycle_ptr, x.cycle_edges.cpu().tolist()))
    assert got[0] == got[1]

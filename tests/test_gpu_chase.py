"""The value chase and the device-driven loop against the round-by-round
path (G lanes per vertex, which keeps it) and the oracle, at the sizes and
values where the chase changes its form: workgroup edges, the scope rule's
limits, passes that do not finish, stalls, and sums beyond the packed entry."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import native
from paper_1111_0627_amd import ocm, synth

pytestmark = pytest.mark.gpu


def both(g, mode="min", t=None):
    dev = [torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in (g.row_ptr, g.col, g.w)]
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
    for r in (a, b):
        assert r.cycle_edges.numel() > 0
    same = ("p", "q", "W", "L", "source", "iterations", "flags", "tight_edges", "fast_iters",
            "connect_rounds")
    assert [getattr(a, k) for k in same] == [getattr(b, k) for k in same]
    for k in ("cycle_edges", "policy", "potential"):
        assert torch.equal(getattr(a, k), getattr(b, k)), k
    return a


@pytest.mark.parametrize("n", [1, 2, 5, 255, 256, 257, 4095, 4097, 65537, (1 << 17) - 1, 1 << 17,
                               (1 << 18) - 1, 1 << 18, 300007])
def test_sizes(n, monkeypatch):
    monkeypatch.setenv("OCM_SMALL", "0")
    g = synth.random_digraph(n, 1, 4, -1000, 1000, np.int64, seed=[71, n])
    r = both(g, "min" if n % 2 else "max")
    if n <= 4095:
        sol = native.solve(g.row_ptr, g.col, g.w, "min" if n % 2 else "max")
        assert (r.p, r.q, r.iterations, r.cycle_edges.cpu().tolist()) == \
            (sol.p, sol.q, sol.iterations, sol.cycle.tolist())


@pytest.mark.parametrize("n", [257, 20011])
def test_times(n, monkeypatch):
    monkeypatch.setenv("OCM_SMALL", "0")
    g = synth.random_digraph(n, 1, 5, -500, 500, np.int32, seed=[72, n])
    t = np.random.default_rng(n).integers(1, 20, g.m).astype(np.int32)
    both(g, "max" if n == 257 else "min", t)


@pytest.mark.parametrize("seed", range(4))
def test_small_weights_stall_and_tie(seed, monkeypatch):
    monkeypatch.setenv("OCM_SMALL", "0")
    """Few distinct weights: policy cycles away from C (stalls), ties."""
    g = synth.random_digraph(5000, 1, 4, 0, 2, np.int32, seed=[73, seed])
    both(g)


def test_long_paths_take_several_passes():
    """A ring of n vertices with one heavy shortcut: paths of n - 1 edges."""
    n = 70000
    rp = np.arange(n + 1, dtype=np.int32)
    col = ((np.arange(n) + 1) % n).astype(np.int32)
    w = np.random.default_rng(5).integers(-50, 50, n)
    rp[1:] += 1                       # vertex 0: a second edge, to vertex 1
    col = np.insert(col, 1, 1).astype(np.int32)
    w = np.insert(w, 1, 40).astype(np.int64)
    g = synth.Graph(rp, col, w, "ring")
    r = both(g)
    assert r.cycle_edges.numel() == n


@pytest.mark.parametrize("hlo", [2**22, 2**35, 2**47])
def test_sums_beyond_the_entry(hlo, monkeypatch):
    """Sums of 2^22, of more than the entry's 53 bits, and beyond int64."""
    monkeypatch.setenv("OCM_SMALL", "0")
    g = synth.deep_tail_graph(700, 800, 2, 10, hlo, 2 * hlo, seed=3)
    dev = [torch.from_numpy(x).cuda() for x in (g.row_ptr, g.col, g.w)]
    r = ocm.min_cycle_mean(*dev)
    sol = native.solve(g.row_ptr, g.col, g.w)
    assert (r.p, r.q, r.iterations, r.cycle_edges.cpu().tolist()) == \
        (sol.p, sol.q, sol.iterations, sol.cycle.tolist())
    assert r.int128 == (hlo == 2**47)
    if hlo < 2**47:
        both(g)


@pytest.mark.parametrize("hubs,deg", [(1, 100), (3, 33), (2, 9000)])
def test_rebuild_rounds_over_long_rows(hubs, deg):
    """Rows around the whole-wave limit and beyond the giant-row limit."""
    both(synth.hub_graph(9000, hubs, deg, 1, 3, -20, 20, np.int64, seed=[76, deg]))


def test_disconnected(monkeypatch):
    monkeypatch.setenv("OCM_SMALL", "0")
    for n in (6000, 1 << 17):
        v = np.arange(n)
        col = np.where(v % (n // 2) == n // 2 - 1, v - (n // 2 - 1), v + 1).astype(np.int32)
        dev = [torch.from_numpy(x).cuda() for x in (np.arange(n + 1, dtype=np.int32), col, (v < n // 2).astype(np.int32))]
        for sched in (0, 8):
            with pytest.raises(ocm.OCMError) as e:
                ocm.min_cycle_mean(*dev, schedule=sched)
            assert e.value.status == ocm.OCM_E_NOT_STRONGLY_CONNECTED


def test_values_leave_int32_in_mid_solve():
    """int64 weights whose values do not fit the int32 copy."""
    g = synth.random_digraph(20000, 1, 5, 2**30, 2**31, np.int64, seed=[74, 0])
    both(g)


def batch(gs, mode="min", **kw):
    u, vptr, eptr = synth.disjoint_union(gs)
    dev = [torch.from_numpy(x).cuda() for x in (u.row_ptr, u.col, u.w)]
    r = ocm.cycle_mean_batched(*dev, vptr, eptr, mode=mode, **kw)
    return r, [tuple(e - int(eptr[k]) for e in r.cycle(k).cpu().tolist()) for k in range(len(gs))]


def check_batch(gs, mode="min"):
    """The loop's chase against its rounds (G lanes per vertex) and the oracle."""
    (a, ca), (b, cb) = batch(gs, mode), batch(gs, mode, schedule=4)
    for k in ("p", "q", "iterations", "flags", "status", "cycle_ptr"):
        assert getattr(a, k) == getattr(b, k), k
    assert ca == cb
    for k, g in enumerate(gs):
        if a.status[k] != ocm.OCM_OK:
            continue
        sol = native.solve(g.row_ptr, g.col, g.w, mode)
        assert (a.p[k], a.q[k], a.iterations[k], list(ca[k])) == \
            (sol.p, sol.q, sol.iterations, sol.cycle.tolist())
    return a


@pytest.mark.parametrize("sizes", [[1, 2, 3], [255, 256, 257], [511, 512, 513, 1025], [20011, 1, 4097]])
def test_batched_loop_sizes(sizes, monkeypatch):
    monkeypatch.setenv("OCM_BATCH_SMALL", "0")
    monkeypatch.setenv("OCM_BATCH_SOLO", "0")
    check_batch([synth.random_digraph(n, 1, 4, -100, 100, np.int64, seed=[81, n]) for n in sizes],
                "max" if len(sizes) == 3 else "min")


@pytest.mark.parametrize("sizes", [[1], [5000], [2, 30000, 257, 6000], [100, 4000, 200, 7000, 300]])
def test_few_large_graphs_solved_alone(sizes, monkeypatch):
    """At most four graphs beyond the small class leave the loop; failing ones
    keep the batch's statuses."""
    gs = [synth.random_digraph(n, 1, 4, -100, 100, np.int64, seed=[84, n]) for n in sizes]
    if len(sizes) == 5:
        gs.append(synth.deep_tail_graph(700, 1500, 2, 10, 2**47, 2**48, seed=3))
        n = 6000                            # two rings
        v = np.arange(n)
        col = np.where(v % 3000 == 2999, v - 2999, v + 1).astype(np.int32)
        gs.append(synth.Graph(np.arange(n + 1, dtype=np.int32), col, (v < 3000).astype(np.int64), "rings"))
    got = []
    for solo in ("1", "0"):
        monkeypatch.setenv("OCM_BATCH_SOLO", solo)
        if len(sizes) == 1:
            monkeypatch.setenv("OCM_BATCH_SMALL", "0")
        r = check_batch(gs, "max" if len(sizes) == 4 else "min")
        got.append((r.p, r.q, r.flags, r.status, r.cycle_ptr, r.cycle_edges.cpu().tolist(),
                    r.iterations))
    assert got[0] == got[1]
    if len(sizes) == 5:
        assert got[0][3] == [0] * 5 + [ocm.OCM_E_OVERFLOW, ocm.OCM_E_NOT_STRONGLY_CONNECTED]


def test_batched_stalls_and_ties(monkeypatch):
    monkeypatch.setenv("OCM_BATCH_SMALL", "0")
    monkeypatch.setenv("OCM_BATCH_SOLO", "0")
    check_batch([synth.random_digraph(3000 + k, 1, 4, 0, 2, np.int64, seed=[82, k]) for k in range(8)])


@pytest.mark.parametrize("hlo", [2**35, 2**47])
def test_batched_sums_beyond_the_entry(hlo, monkeypatch):
    """A graph whose sums do not fit the packed entries goes on with the
    doubling rounds; one beyond int64 fails alone."""
    monkeypatch.setenv("OCM_BATCH_SMALL", "0")
    monkeypatch.setenv("OCM_BATCH_SOLO", "0")
    gs = [synth.random_digraph(n, 1, 5, 1, 1000, np.int64, seed=[83, n]) for n in (300, 5000)]
    gs.insert(1, synth.deep_tail_graph(700, 800, 2, 10, hlo, 2 * hlo, seed=3))
    r = check_batch(gs)
    assert r.status == [0, ocm.OCM_E_OVERFLOW if hlo == 2**47 else 0, 0]


def test_batched_long_paths(monkeypatch):
    """Rings of n vertices with a shortcut: paths of n - 1 edges, cycles of n."""
    monkeypatch.setenv("OCM_BATCH_SMALL", "0")
    monkeypatch.setenv("OCM_BATCH_SOLO", "0")
    gs = []
    for n in (3000, 70000):
        col = np.insert((np.arange(n) + 1) % n, 1, 1).astype(np.int32)
        rp = np.arange(n + 1, dtype=np.int32)
        rp[1:] += 1
        w = np.insert(np.random.default_rng(n).integers(-50, 50, n), 1, 40).astype(np.int64)
        gs.append(synth.Graph(rp, col, w, "ring"))
    check_batch(gs)


@pytest.mark.parametrize("cap", [1, 2, 3, 5])
def test_iteration_cap(cap, monkeypatch):
    monkeypatch.setenv("OCM_SMALL", "0")
    g = synth.random_digraph(3000, 1, 4, 1, 1000, np.int32, seed=[75, 0])
    dev = [torch.from_numpy(x).cuda() for x in (g.row_ptr, g.col, g.w)]
    need = ocm.min_cycle_mean(*dev).iterations
    assert need > 5
    for sched in (0, 8):
        with pytest.raises(ocm.OCMError) as e:
            ocm.min_cycle_mean(*dev, max_iters=cap, schedule=sched)
        assert e.value.status == ocm.OCM_E_NOT_CONVERGED
    assert ocm.min_cycle_mean(*dev, max_iters=need).iterations == need


@pytest.mark.parametrize("a,b,whi", [(640, 512, 1000), (2100, 150, 1000), (700, 640, 3)])
def test_deep_policies_in_passes_of_few_steps(a, b, whi):
    """Tori of at least 2^18 vertices: most paths take hundreds of edges, so that
    waves stop early from the second value phase on."""
    n = a * b
    v = np.arange(n)
    col = np.stack([(v % a + 1) % a + v // a * a, v % a + (v // a + 1) % b * a], 1)
    w = np.random.default_rng([75, a]).integers(1, whi + 1, (n, 2))
    both(synth.Graph(2 * np.arange(n + 1, dtype=np.int32), col.astype(np.int32).reshape(-1), w.astype(np.int64).reshape(-1)),
         "max" if whi == 3 else "min")

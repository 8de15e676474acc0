"""Rebuild rounds whose direction changes: a pull first and pushes after it, and
warm starts that leave many vertices to attach.  Results are those of the
pull-only rounds; the in-edge counts say that pushes ran."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1111_0627_amd import ocm

pytestmark = pytest.mark.gpu


def layers(near, far, width):
    """`near` vertices lead to the light loop at 0 by a tree, `far` ones keep a
    loop of their own as their first policy and attach `width` per round."""
    v = np.arange(near + far)
    rp = 2 * np.arange(near + far + 1)
    col = np.repeat(v, 2)
    w = np.empty((near + far, 2), np.int64)
    w[:] = 0, 7
    col[1::2] = np.where(v < near, v // 2, np.where(v < near + width, v % near, v - width))
    w[:near, 0] = 9
    w[0] = -10, 5
    i32 = np.int32
    return [torch.from_numpy(x).cuda() for x in (rp.astype(i32), col.astype(i32), w.astype(i32).reshape(-1))]


def same(a, b):
    for k in ("p", "q", "W", "L", "source", "iterations", "flags", "tight_edges", "connect_rounds"):
        assert getattr(a, k) == getattr(b, k), k
    for k in ("cycle_edges", "policy", "potential"):
        assert torch.equal(getattr(a, k), getattr(b, k)), k


WHOLE = dict(want_policy=True, want_potential=True)


@pytest.mark.parametrize("near,far,width", [(300_000, 140_000, 1000), (200_000, 131_072, 997), (1 << 18, 200_001, 4096)])
def test_pushes_after_a_pull(near, far, width):
    """2 * near >= far: the first round pulls and leaves no marks to the pushes behind it."""
    g = layers(near, far, width)
    a = ocm.min_cycle_mean(*g, **WHOLE)
    same(a, ocm.min_cycle_mean(*g, connect="pull", **WHOLE))
    assert a.connect_rounds >= far // width
    # every in-edge of the layers attached while more than 65,536 vertices are left
    assert a.counters["push_in_edges"] >= far - 65536 - 2 * width


def test_warm_start_with_millions_left():
    near, far, width = 300_000, (1 << 22) + 200_001, 100_003
    g = layers(near, far, width)
    policy = 2 * torch.arange(near + far, device="cuda", dtype=torch.int32)
    policy[1:near] += 1
    a = ocm.min_cycle_mean(*g, init_policy=policy, **WHOLE)
    same(a, ocm.min_cycle_mean(*g, init_policy=policy, connect="pull", **WHOLE))
    assert a.connect_rounds >= far // width
    assert a.counters["push_in_edges"] > 0


def test_warm_start_with_some_left():
    near, far, width = 150_000, 100_000, 1000
    g = layers(near, far, width)
    policy = 2 * torch.arange(near + far, device="cuda", dtype=torch.int32)
    policy[1:near] += 1
    for n_far in (far, 0):
        if n_far == 0:
            policy[near:] += 1   # everybody reaches C
        a = ocm.min_cycle_mean(*g, init_policy=policy, **WHOLE)
        same(a, ocm.min_cycle_mean(*g, init_policy=policy, connect="pull", **WHOLE))

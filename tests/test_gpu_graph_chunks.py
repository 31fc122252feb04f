"""Calls of every small number of steps replay graphs of 8, 4, 2 and 1 steps from either state
buffer; a batch's launch groups run in lanes of their own.  Every result is bitwise that of eager
launches, call after call, with other eager work between the replays."""
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

CALLS = [1, 2, 3, 1, 1, 5, 7, 8, 15, 3]


@pytest.fixture(scope="module")
def dg():
    from paper_2206_09733_amd import dgsem
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    dgsem.lib()
    return dgsem


def make(dg, scheme, graphs, **kw):
    s = dg.Solver(**kw)
    s.set_scheme(scheme)
    s.use_graphs(graphs)
    s.set_ic("tgv")
    return s


@pytest.mark.parametrize("scheme", ["rk3", "rk4"])
def test_solver_graph_chunks(dg, scheme):
    import torch
    print("graph chunks", scheme, flush=True)
    kw = dict(ex=3, ey=2, ez=3, N=3, deform=True, Ma=0.2, Re=100.0)
    a, b = make(dg, scheme, True, **kw), make(dg, scheme, False, **kw)
    for n in CALLS:
        a.rk_step(1e-3, n)
        torch.ones(1000, device="cuda").sum().item()
        b.rk_step(1e-3, n)
        assert np.array_equal(a.state(), b.state()), n
    a.close()
    b.close()


@pytest.mark.parametrize("scheme", ["rk3", "rk4"])
def test_batch_graph_chunks(dg, scheme):
    """Six launch groups and a mixed-order member: more units than lanes."""
    import torch
    from paper_2206_09733_amd import synth
    print("batch graph chunks", scheme, flush=True)
    kws = [dict(ex=2, ey=3, ez=1 + i % 3, N=2 + i % 3, Ma=0.2, Re=100.0 * (i % 2), deform=i == 4) for i in range(9)]
    kws.append(dict(ex=2, orders=synth.mixed_orders(8, seed=1), Ma=0.5))
    sets = [[make(dg, scheme, g, **k) for k in kws] for g in (True, False)]
    A, B = dg.Batch(sets[0]), dg.Batch(sets[1])
    B.use_graphs(False)
    dts = [1e-3 * (1 + 0.1 * i) for i in range(len(kws))]
    for n in CALLS:
        A.rk_step(dts, n)
        torch.ones(1000, device="cuda").sum().item()
        B.rk_step(dts, n)
        for x, y in zip(*sets):
            assert np.array_equal(x.state(), y.state()), n
    A.close()
    B.close()
    for s in sets[0] + sets[1]:
        s.close()
    sys.stdout.flush()


def test_batch_steps_under_a_callers_capture(dg):
    """Eager batch steps captured by the caller: the launches of every lane are one chain of the
    captured stream, and each replay advances the members as eager steps do."""
    import torch
    print("batch under a caller's capture", flush=True)
    kws = [dict(ex=2, ey=3, ez=1 + i % 3, N=2 + i % 3, Ma=0.2, Re=100.0 * (i % 2)) for i in range(6)]
    sets = [[make(dg, "rk3", False, **k) for k in kws] for _ in range(2)]
    dts = [1e-3 * (1 + 0.1 * i) for i in range(len(kws))]
    side = torch.cuda.Stream()
    A, B = dg.Batch(sets[0], stream=side), dg.Batch(sets[1])
    A.use_graphs(False)
    B.use_graphs(False)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=side):
        A.rk_step(dts, 2)  # an even number of stages: the state returns to its buffer
    for _ in range(3):
        g.replay()
        torch.ones(1000, device="cuda").sum().item()
        torch.cuda.synchronize()
        B.rk_step(dts, 2)
        for x, y in zip(*sets):
            assert np.array_equal(x.state(), y.state())
    A.close()
    B.close()
    for s in sets[0] + sets[1]:
        s.close()

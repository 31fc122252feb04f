"""The stage kernel's forms against the oracle, at the sizes where each can go wrong: plain boxes
(constant metric terms, fluxes in rotated frames) and deformed ones at every order, low orders that
pack several elements into a workgroup with a remainder, and node-to-node jumps on both sides of
each tier of the logarithmic mean (relative differences of 1%, 20% and ratios up to hundreds).  The
bar is the parity gate (GATE times the FP64 oracle's distance to the long-double oracle, or 1e-12
relative); FP32-bulk at its stated tolerance.
"""
import sys

import numpy as np
import pytest

from helpers import FP32_TOL, GATE, gate_ok, rel_per_var

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dg():
    from paper_2206_09733_amd import dgsem
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    dgsem.lib()
    return dgsem


def log(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def random_state(E, nn, seed, ratio):
    """rho and p independent at every node, log-uniform in [1/ratio, ratio]; |v| up to 0.5."""
    g = np.random.Generator(np.random.PCG64(seed))
    rho, p = np.exp(g.uniform(-1, 1, (2, E, nn)) * np.log(ratio))
    v = g.uniform(-0.5, 0.5, (3, E, nn))
    return np.stack([rho, *(rho * v), p / 0.4 + 0.5 * rho * (v * v).sum(0)], 1).reshape(-1)


def check(dg, orc, name, c, U, E, nn):
    log(name, c)
    g = dg.Solver(**c)
    g.set_state(U)
    G = g.residual().reshape(E, 5, nn)
    g.close()
    R = []
    for prec in ("fp64", "fp80"):
        o = orc.OracleSolver(**c, precision=prec)
        o.set_state(U)
        R.append(o.residual().reshape(E, 5, nn))
    scale = np.abs(R[1]).max(axis=(0, 2))
    e64 = np.abs(R[0] - R[1]).max(axis=(0, 2))
    eg = np.abs(G - R[1]).max(axis=(0, 2))
    log(f"gpu-vs-fp80={eg / scale} fp64-vs-fp80={e64 / scale}")
    assert gate_ok(name, eg, e64, scale), (name, eg, np.maximum(1e-12 * scale, GATE * e64))


@pytest.mark.parametrize("deform", [False, True])
@pytest.mark.parametrize("N", [1, 2, 3, 4, 5, 6, 7])
@pytest.mark.parametrize("vol,surf,Re", [("ec", "roe", 0.0), ("ec", "ec", 50.0), ("central", "llf", 50.0),
                                         ("ir", "es_matrix", 0.0), ("pirozzoli", "ld_roe", 50.0)])
def test_stage_forms(dg, orc, N, deform, vol, surf, Re):
    """15 elements: no multiple of a workgroup's 8 (N = 1) or 2 (N = 2), nor of the 8 XCDs."""
    c = dict(ex=3, ey=1, ez=5, deform=deform, N=N, Ma=0.5, Re=Re, vol=vol, surf=surf)
    if not deform:  # (the deformation has period 2 pi)
        c["hi"] = (1.0, 0.5, 2.0)
    check(dg, orc, f"forms {vol}+{surf}", c, random_state(15, (N + 1) ** 3, 11 * N, 1.3), 15, (N + 1) ** 3)


@pytest.mark.parametrize("ratio", [1.01, 1.2, 30.0])
@pytest.mark.parametrize("vol,surf", [("ec", "ec"), ("ir", "ir"), ("ec", "es_matrix")])
def test_logarithmic_mean_tiers(dg, orc, ratio, vol, surf):
    c = dict(ex=3, ey=2, ez=1, N=3, Ma=0.5, vol=vol, surf=surf)
    check(dg, orc, f"log-mean tiers {vol}+{surf} {ratio}", c, random_state(6, 64, 5, ratio), 6, 64)


@pytest.mark.parametrize("deform", [False, True])
@pytest.mark.parametrize("N", [1, 2, 3, 4, 5, 6, 7])
@pytest.mark.parametrize("vol,surf,Re", [("ec", "roe", 0.0), ("central", "llf", 200.0), ("ec", "ec", 200.0)])
def test_stage_forms_fp32_bulk(dg, orc, N, deform, vol, surf, Re):
    c = dict(ex=3, ey=5, ez=3, N=N, deform=deform, Ma=0.1, Re=Re, vol=vol, surf=surf)
    log(f"fp32 forms {c}")
    o = orc.OracleSolver(**c)
    o.set_ic("tgv")
    g = dg.Solver(**c, precision="fp32_bulk")
    g.set_state(o.state())
    err = rel_per_var(g.residual(), o.residual(), 45)
    g.close()
    log(err)
    assert np.all(err <= FP32_TOL["small"]), err


@pytest.mark.parametrize("fp32", [False, True])
@pytest.mark.parametrize("N", [1, 2, 4])
def test_batch_of_plain_and_deformed_boxes(dg, N, fp32):
    """A batch whose members are all plain, and one that mixes plain and deformed boxes, of odd
    element counts: every member bitwise as when it is stepped alone."""
    for boxes in ((False, False, False), (False, True, False)):
        kw = [dict(ex=3, ey=1, ez=5 - 2 * i, N=N, deform=b, Ma=0.2, Re=100.0 * (1 + i),
                   precision="fp32_bulk" if fp32 else "fp64") for i, b in enumerate(boxes)]
        log(f"batch {kw}")
        ref, mem = [], []
        for k in kw:
            for out in (ref, mem):
                s = dg.Solver(**k)
                s.set_ic("tgv")
                out.append(s)
        for s in ref:
            s.rk_step(1e-3, 3)
        b = dg.Batch(mem)
        assert b.launches_per_stage() == 2
        b.rk_step([1e-3] * 3, 3)
        for r, m in zip(ref, mem):
            assert np.array_equal(r.state(), m.state())
        b.close()
        for s in ref + mem:
            s.close()


@pytest.mark.parametrize("N,box", [(1, (7, 16, 16)), (1, (7, 16, 17)), (2, (5, 3, 3)), (2, (9, 10, 21)), (3, (3, 3, 3)),
                                   (3, (14, 8, 8)), (4, (2, 3, 3)), (4, (9, 11, 7))])
@pytest.mark.parametrize("fp32,Re,deform", [(False, 0.0, True), (False, 100.0, False), (True, 0.0, True), (True, 100.0, False)])
def test_small_mesh_shape(dg, N, box, fp32, Re, deform):
    """Meshes up to 1792 waves step alone in the small launch shape and as members of a batch in the
    usual one: the states are bitwise the same, below, at and above the line."""
    c = dict(ex=box[0], ey=box[1], ez=box[2], N=N, Re=Re, deform=deform, Ma=0.3,
             precision="fp32_bulk" if fp32 else "fp64")
    log("small shape", c)
    S = [dg.Solver(**c) for _ in range(3)]
    for s in S:
        s.set_ic("tgv")
    S[0].rk_step(1e-3, 3)
    b = dg.Batch(S[1:])
    b.rk_step([1e-3] * 2, 3)
    U = [s.state() for s in S]
    b.close()
    for s in S:
        s.close()
    assert np.isfinite(U[0]).all()
    assert np.array_equal(U[0], U[1]) and np.array_equal(U[0], U[2])


@pytest.mark.parametrize("tiles", [0, 63])
@pytest.mark.parametrize("deform", [False, True])
@pytest.mark.parametrize("vol,surf", [("ec", "roe"), ("central", "llf"), ("ir", "es"), ("kg", "es_matrix")])
def test_mixed_stage_forms(dg, orc, vol, surf, deform, tiles):
    """Per-element orders 1..6 (every cyclic distance and both parities of the node count), plain and
    deformed boxes, one and two nodes per lane."""
    from paper_2206_09733_amd import synth
    c = dict(ex=3, ey=2, ez=5, orders=synth.mixed_orders(30, seed=4, lo=1, hi=6), deform=deform, Ma=0.5, vol=vol,
             surf=surf)
    log(f"mixed forms {vol} {surf} {deform} {tiles}")
    o80 = orc.OracleSolver(**c, precision="fp80")
    o64 = orc.OracleSolver(**c)
    g = np.random.Generator(np.random.PCG64(7))
    U = []
    for a in np.asarray(c["orders"]).reshape(-1, 3):
        nn = int(np.prod(a + 1))
        rho, p = np.exp(g.uniform(-1, 1, (2, nn)) * np.log(1.3))
        v = g.uniform(-0.5, 0.5, (3, nn))
        U.append(np.concatenate([rho, *(rho * v), p / 0.4 + 0.5 * rho * (v * v).sum(0)]))
    U = np.concatenate(U)
    for o in (o64, o80):
        o.set_state(U)
    s = dg.Solver(**c)
    s.set_tiles(tiles)
    s.set_state(U)
    G, A, B = s.residual(), o64.residual(), o80.residual()
    s.close()
    scale, e64, eg = np.abs(B).max(), np.abs(A - B).max(), np.abs(G - B).max()
    log(eg / scale, e64 / scale)
    assert gate_ok(f"mixed forms {vol}+{surf}", [eg], [e64], [scale])

"""Every form of the batched stage and gradient kernels against the same solver stepped alone: bitwise
the same states, whatever launch shape either of them takes (a small mesh alone runs one element per
workgroup, and so does order 1 in a small batch; otherwise orders 1 and 2 are packed, with a remainder
here: 15 elements in workgroups of 2, 2028 in workgroups of 8).  The solvers alone are checked against
the oracle elsewhere."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

FLUXES = [("ec", "roe"), ("central", "llf"), ("ec", "ec"), ("ec", "es"), ("ir", "es_matrix"), ("kg", "ld_roe"),
          ("kg", "es_matrix"), ("pirozzoli", "lf_global")]
VISCOUS = [dict(), dict(Re=50.0), dict(Re=50.0, visc="br2"), dict(Re=50.0, visc="ip")]


@pytest.fixture(scope="module")
def dg():
    from paper_2206_09733_amd import dgsem
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    dgsem.lib()
    return dgsem


def random_state(E, nn, seed):
    """rho and p independent at every node, log-uniform in [1/1.3, 1.3]; |v| up to 0.5."""
    g = np.random.Generator(np.random.PCG64(seed))
    rho, p = np.exp(g.uniform(-1, 1, (2, E, nn)) * np.log(1.3))
    v = g.uniform(-0.5, 0.5, (3, E, nn))
    return np.stack([rho, *(rho * v), p / 0.4 + 0.5 * rho * (v * v).sum(0)], 1).reshape(-1)


def compare(dg, boxes, steps=2, **c):
    """Members on `boxes` = (cells, deform, hi) in one batch, each against itself alone."""
    print("batch forms", boxes, c, flush=True)
    alone, batched = [], []
    for i, (cells, deform) in enumerate(boxes):
        E, nn = int(np.prod(cells)), (c["N"] + 1) ** 3
        kw = dict(c, ex=cells[0], ey=cells[1], ez=cells[2], deform=deform, Ma=0.5)
        if not deform:  # (the deformation has period 2 pi)
            kw["hi"] = (1.0, 0.5, 2.0)
        U = random_state(E, nn, 17 * c["N"] + i)
        for out in (alone, batched):
            out.append(dg.Solver(**kw))
            out[-1].set_state(U)
            out[-1].use_graphs(False)
    b = dg.Batch(batched)
    b.use_graphs(False)
    b.rk_step([1e-5] * len(batched), steps)
    for k, (x, y) in enumerate(zip(alone, batched)):
        x.rk_step(1e-5, steps)
        A, B = x.state(), y.state()
        assert np.isfinite(A).all()
        assert np.array_equal(A, B), (k, np.abs(A - B).max())
    b.close()
    for s in alone + batched:
        s.close()


@pytest.mark.parametrize("N", [1, 2, 3, 4, 5, 6, 7])
@pytest.mark.parametrize("vol,surf", FLUXES)
def test_batch_forms_equal_alone(dg, N, vol, surf):
    for visc in VISCOUS:
        for deform in (False, True):
            compare(dg, [((3, 1, 5), deform), ((3, 1, 5), deform)], N=N, vol=vol, surf=surf, **visc)


@pytest.mark.parametrize("N", [1, 2, 3, 4, 5, 6, 7])
@pytest.mark.parametrize("vol,surf", [("ec", "roe"), ("central", "llf"), ("ec", "ec"), ("central", "central")])
def test_fp32_bulk_batch_forms_equal_alone(dg, N, vol, surf):
    for visc in VISCOUS:
        for deform in (False, True):
            compare(dg, [((3, 1, 5), deform), ((3, 1, 5), deform)], N=N, vol=vol, surf=surf, precision="fp32_bulk",
                    **visc)


@pytest.mark.parametrize("precision", ["fp64", "fp32_bulk"])
@pytest.mark.parametrize("N", [1, 2, 3, 4, 5, 6, 7])
def test_plain_and_deformed_members_equal_alone(dg, N, precision):
    for visc in VISCOUS:
        compare(dg, [((3, 1, 5), False), ((2, 3, 3), True), ((1, 1, 1), False)], N=N, precision=precision, **visc)
    if N == 1:  # packed: 8 elements per workgroup, a remainder in each member
        for visc in VISCOUS:
            compare(dg, [((9, 10, 9), False), ((7, 11, 13), True)], N=N, precision=precision, **visc)


@pytest.mark.parametrize("N,cells", [(1, (13, 12, 13)), (1, (17, 15, 13)), (2, (13, 12, 13)), (3, (9, 10, 11)), (4, (9, 9, 9))])
@pytest.mark.parametrize("vol,surf", FLUXES)
def test_batch_forms_equal_alone_above_the_small_shape(dg, N, cells, vol, surf):
    """Meshes that take the usual shape alone and in the batch (order 1: 8 elements per workgroup)."""
    for visc in VISCOUS:
        for deform in (False, True):
            compare(dg, [(cells, deform)], steps=1, N=N, vol=vol, surf=surf, **visc)

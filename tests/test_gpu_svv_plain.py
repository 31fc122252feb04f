"""Spectral vanishing viscosity and the LES closures on plain boxes (constant metric terms, none read), every
order, against the oracle: FP64 at the parity gate, FP32-bulk at its stated tolerance."""
import numpy as np
import pytest

from helpers import FP32_TOL
from test_gpu_svv import gpu_solver, log, oracles, parity, perturbed

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dg():
    from paper_2206_09733_amd import dgsem
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    dgsem.lib()
    return dgsem


@pytest.mark.parametrize("N", [1, 2, 3, 4, 5, 6, 7])
@pytest.mark.parametrize("kernel,extra", [("maday", dict()), ("tadmor", dict(Re=200.0)),
                                          ("maday", dict(Re=200.0, visc="br2")), ("tadmor", dict(Re=200.0, surf="es"))])
def test_plain_svv_residual_parity(dg, orc, N, kernel, extra):
    c = dict(ex=3, ey=2, ez=4, N=N, Ma=0.3, **extra)
    svv = dict(mu=0.02, kernel=kernel, cutoff=N // 2)
    log(f"plain svv {c} {kernel}")
    U = perturbed(orc, c, seed=2200 + N)
    o64, o80 = oracles(orc, c, U, svv)
    g = gpu_solver(dg, c, svv)
    g.set_state(U)
    parity(f"plain svv N={N} {kernel} {extra}", g.residual(), o64.residual(), o80.residual(), 24, (N + 1) ** 3)
    g.close()


@pytest.mark.parametrize("N", [1, 2, 3, 4, 5, 6, 7])
@pytest.mark.parametrize("Re", [0.0, 1600.0])
@pytest.mark.parametrize("les", [None, ("wale", 0.5)])
def test_plain_svv_fp32_bulk_residual(dg, orc, N, Re, les):
    c = dict(ex=3, ey=4, ez=3, N=N, Ma=0.1, Re=Re)
    log(f"plain svv fp32 {c} {les}")
    o = orc.OracleSolver(**c)
    if les:
        o.set_les(les[1], les[0])
    o.set_svv(0.02, "maday", N // 2, -1.0)
    o.set_ic("tgv")
    extra = dict(les_cs=les[1], les_model=les[0]) if les else {}
    g = dg.Solver(**c, svv_mu=0.02, svv_kernel="maday", svv_cutoff=N // 2, precision="fp32_bulk", **extra)
    g.set_state(o.state())
    G, R = (x.reshape(36, 5, -1) for x in (g.residual(), o.residual()))
    g.close()
    err = np.abs(G - R).max(axis=(0, 2)) / np.abs(R).max(axis=(0, 2))
    log(err)
    assert np.all(err < FP32_TOL["small"]), err

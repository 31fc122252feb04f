"""The logarithmic means at large ratios of the two nodes' values, and at values they have no meaning for."""
import numpy as np
import pytest

from helpers import gate_ok

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dg():
    from paper_2206_09733_amd import dgsem
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    dgsem.lib()
    return dgsem


@pytest.mark.parametrize("deform", [False, True])
@pytest.mark.parametrize("ratio", [1e4, 1e8, 1e12, 1e16, 1e22, 1e30, 1e40])
@pytest.mark.parametrize("vol,surf", [("ec", "ec"), ("ir", "ir")])
def test_logarithmic_mean_of_large_ratios(dg, orc, ratio, vol, surf, deform):
    """Every node's density is 1 or 1/ratio (p = 1), |v| up to 0.5: the fluxes between the two kinds carry
    1/ln(ratio) of the largest ones, so an error of the mean shows at 1/30 to 1/100 of itself.  The bar
    per variable: the parity gate with 1e-13 of the largest residual as its floor, a thousand roundings."""
    N, E, nn = 3, 6, 64
    g = np.random.Generator(np.random.PCG64(3))
    rho = np.where(g.random((E, nn)) < 0.5, 1.0, 1.0 / ratio)
    v = g.uniform(-0.5, 0.5, (3, E, nn))
    U = np.stack([rho, *(rho * v), 2.5 + 0.5 * rho * (v * v).sum(0)], 1).reshape(-1)
    c = dict(ex=3, ey=2, ez=1, N=N, Ma=0.5, vol=vol, surf=surf, deform=deform)
    print("log mean", vol, surf, ratio, deform, flush=True)
    s = dg.Solver(**c)
    s.set_state(U)
    G = s.residual().reshape(E, 5, nn)
    s.close()
    R = []
    for prec in ("fp64", "fp80"):
        o = orc.OracleSolver(**c, precision=prec)
        o.set_state(U)
        R.append(o.residual().reshape(E, 5, nn))
    scale = np.abs(R[1]).max(axis=(0, 2))
    e64, eg = (np.abs(x - R[1]).max(axis=(0, 2)) for x in (R[0], G))
    print(eg / scale, e64 / scale, flush=True)
    assert np.isfinite(G).all()
    assert gate_ok(f"log mean {vol}+{surf} {ratio}", eg, e64, scale, floor=1e-13)


@pytest.mark.parametrize("precision", ["fp64", "fp32_bulk"])
@pytest.mark.parametrize("N", [2, 4])
def test_negative_densities_do_not_pass_as_finite(dg, N, precision):
    """Two nodes of negative density whose values differ have no logarithmic mean: the residual of an
    element of such nodes is not finite."""
    nn = (N + 1) ** 3
    s = dg.Solver(ex=3, ey=3, ez=3, N=N, Ma=0.5, vol="ec", surf="central", precision=precision)
    s.set_ic("uniform", [1.0, 0.1, 0.2, 0.3, 1.0])
    off = s.device_pointers()[0] - s.buf.data_ptr()
    import torch
    U = s.buf[off:off + 40 * s.nodes].view(torch.float64).view(27, 5, nn)
    g = torch.Generator().manual_seed(1)
    U[13, 0] = -(1.0 + 2.0 * torch.rand(nn, generator=g, dtype=torch.float64)).to(U.device)
    torch.cuda.synchronize()
    R = s.residual().reshape(27, 5, nn)
    s.close()
    print("negative densities", N, precision, np.isfinite(R[13]).mean(), flush=True)
    assert not np.isfinite(R[13, 0]).any()

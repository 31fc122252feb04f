"""The graphs a batch keeps: a member whose captured launches hold values of its own (the FP32-bulk
reference state of a mixed-order or filtered member) replays none that was captured before those
values changed."""
import numpy as np
import pytest

from paper_2206_09733_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dg():
    from paper_2206_09733_amd import dgsem
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    dgsem.lib()
    return dgsem


FP32_SOLO = {
    "mixed": dict(ex=2, orders=synth.mixed_orders(8, seed=1), Ma=0.5, precision="fp32_bulk"),
    "svv": dict(ex=2, N=4, Ma=0.3, Re=100.0, svv_mu=0.01, svv_kernel="maday", svv_cutoff=2, precision="fp32_bulk"),
    "svv_euler": dict(ex=2, N=3, Ma=0.3, svv_mu=0.01, svv_kernel="maday", svv_cutoff=1, precision="fp32_bulk"),
}


@pytest.mark.parametrize("name", list(FP32_SOLO))
def test_replay_after_a_new_state_of_another_mean(dg, name):
    """Replay, a new state of another mean density and pressure in one member, the same steps again:
    bitwise the states of eager launches."""
    print("batch graphs after a new state", name, flush=True)
    other = dict(ex=2, N=3, Ma=0.2)
    sets = [[dg.Solver(**FP32_SOLO[name]), dg.Solver(**other)] for _ in range(2)]
    B = [dg.Batch(s) for s in sets]
    B[1].use_graphs(False)
    for s in sets:
        s[0].set_ic("uniform", [1.0, 0.1, 0.2, 0.3, 2.0])
        s[1].set_ic("tgv")
    for rep, (rho, p) in enumerate(((1.0, 2.0), (2.0, 1.0), (0.5, 3.0))):
        if rep:
            for s in sets:
                s[0].set_ic("density_wave", [0.1, 0.5, 0.2, 0.1, p, 1.0, 1.0, 1.0, 0.1 * rho])
        for n in (2, 3, 2, 1, 1):
            for b in B:
                b.rk_step([1e-3, 1e-3], n)
            for x, y in zip(*sets):
                assert np.array_equal(x.state(), y.state()), (rep, n)
    for b in B:
        b.close()
    for s in sets[0] + sets[1]:
        s.close()

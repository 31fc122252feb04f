"""Calls that only enqueue do not wait for the batch's stream."""
import pytest

pytestmark = pytest.mark.gpu


def test_recurring_step_sizes_replay_without_waiting():
    """Two sets of step sizes, each used in two calls running, of 15 steps: once their graphs are captured
    the calls return while the stream still works on what was enqueued before the first of them."""
    import torch
    from paper_2206_09733_amd import dgsem as dg
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    S = [dg.Solver(ex=2, N=2 + i, Ma=0.2) for i in range(2)]
    for s in S:
        s.set_ic("tgv")
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    b = dg.Batch(S, stream=side)
    cycle = [[1e-3, 1e-3]] * 2 + [[5e-4, 5e-4]] * 2
    for _ in range(3):
        for dts in cycle:
            b.rk_step(dts, 15)
    side.synchronize()
    with torch.cuda.stream(side):
        torch.cuda._sleep(200_000_000)  # 0.08 s to 2 s, by the counter that it reads
        before = torch.cuda.Event()
        before.record(side)
    for k, dts in enumerate(cycle):
        print("call", k, flush=True)
        b.rk_step(dts, 15)
        assert not before.query(), k
    side.synchronize()
    b.close()
    for s in S:
        s.close()

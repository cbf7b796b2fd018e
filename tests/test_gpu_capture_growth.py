"""A caller's capture of a call that may hold cells above 4096 particles, after
eager calls with as many cells but too few particles for one: the large-cell
scratch, fixed in size, is there for it.  Replays against the eager call."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from gpu_helpers import custom_workload


@pytest.mark.parametrize("tangent", [False, True])
def test_capture_after_smaller_calls(tangent):
    import torch
    from paper_2407_19151_amd import native, runner
    ctx = native.Context()
    small = custom_workload([(3, 2)] * 300, seed=1)
    big = custom_workload([(3, 2)] * 296 + [(3000, 2500), (2500, 0), (1200, 300), (5000, 1)],
                          seed=2)

    def call(dw, t):
        if tangent:
            runner.collide_sorted_jvp(ctx, dw, t, 1, update_primal=False)
        else:
            runner.collide_sorted(ctx, dw, 1, with_stats=False)

    def state(wl):
        return runner.DeviceWorkload(wl), torch.ones((3, wl.n), dtype=torch.float64, device="cuda")

    for _ in range(2):
        call(*state(small))
    torch.cuda.synchronize()
    dw, t = state(big)
    start = [x.clone() for x in (dw.vx, dw.vy, dw.vz)]
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        call(dw, t)
    other, want, tw = state(small)[0], *state(big)
    call(want, tw)
    for _ in range(3):
        call(other, torch.ones((3, small.n), dtype=torch.float64, device="cuda"))
        for x, x0 in zip((dw.vx, dw.vy, dw.vz), start):
            x.copy_(x0)
        t.fill_(1.0)
        g.replay()
        torch.cuda.synchronize()
        assert np.array_equal(dw.velocities(), want.velocities()) and bool((t == tw).all())
    assert ctx.device_error() == 0
    assert not bool((tw == 1.0).all()) or not tangent
    ctx.close()


def test_a_graph_keeps_its_scratch():
    """A captured step, then the tangent form, whose scratch is larger, and the
    step on fresh memory: the graph's replay still gives the step's bits."""
    import torch
    from paper_2407_19151_amd import native, runner
    ctx = native.Context()
    wl = custom_workload([(3, 2)] * 20 + [(3000, 2500)], seed=2)
    dw, want = runner.DeviceWorkload(wl), runner.DeviceWorkload(wl)
    runner.collide_sorted(ctx, want, 1, with_stats=False)
    start = [x.clone() for x in (dw.vx, dw.vy, dw.vz)]
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        runner.collide_sorted(ctx, dw, 1, with_stats=False)
    t = torch.ones((3, wl.n), dtype=torch.float64, device="cuda")
    before = torch.cuda.mem_get_info()[0]
    runner.collide_sorted_jvp(ctx, runner.DeviceWorkload(wl), t, 1, update_primal=False)
    torch.cuda.synchronize()
    # (the tangent's large-cell scratch, 4.6 MB a compute unit, in one piece of its own)
    cu = torch.cuda.get_device_properties(0).multi_processor_count
    assert before - torch.cuda.mem_get_info()[0] >= cu * 32768 * 140
    for _ in range(3):
        for x, x0 in zip((dw.vx, dw.vy, dw.vz), start):
            x.copy_(x0)
        g.replay()
        torch.cuda.synchronize()
        assert np.array_equal(dw.velocities(), want.velocities())
    ctx.close()

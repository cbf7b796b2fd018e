"""Size buckets on several streams: a plan (three streams, or two above 2^21
particles) and the per-call step (two above as many cells as compute units)
give the bits of each other over repeated steps; buckets that share the global
scratch against the oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from gpu_helpers import custom_workload
from test_gpu_parity import _parity, ctx  # noqa: F401

# every bucket; two, three and all of them
MIXED = [(40, 30), (100, 90), (200, 150), (400, 300), (700, 600), (1500, 900), (3000, 2500)]


@pytest.mark.parametrize("sizes", [
    MIXED * 3, MIXED * 2 + [(9, 4)] * 400, [(40, 30)] * 200 + [(100, 90)] * 200,
    [(40, 30)] * 200 + [(100, 90)] * 200 + [(200, 150)] * 60,
    [(700, 600)] * 1500 + [(400, 300)] * 300 + [(40, 30)] * 500])
@pytest.mark.parametrize("precision", [0, 1])
def test_plan_and_call_give_the_same_bits(ctx, sizes, precision):  # noqa: F811
    from paper_2407_19151_amd import native, runner
    wl = custom_workload(sizes, seed=17)
    p = runner.params_for(wl, precision=precision)
    dw, dp = runner.DeviceWorkload(wl), runner.DeviceWorkload(wl)
    plan = runner.make_plan(ctx, dp, params=p, autotune=False)
    for step in range(3):
        runner.collide_sorted(ctx, dw, step, params=p)
        plan.run(step, 1)
        if step == 1:
            assert np.array_equal(dp.velocities(), dw.velocities())
    assert np.array_equal(dp.velocities(), dw.velocities())
    assert native.read_stats(dw.stats)["pairs"] > 0
    assert ctx.device_error() == 0
    plan.close()
    assert not np.array_equal(dw.velocities(), wl.velocities())


@pytest.mark.parametrize("pad", [0, 400])
def test_buckets_that_share_the_global_scratch(ctx, pad):  # noqa: F811
    """Three buckets on global-scratch variants (a call's; a plan takes none)."""
    variants = {3: 10, 4: 15, 5: 14}
    for b, v in variants.items():
        ctx.set_variant(b, v)
    try:
        _parity(ctx, custom_workload(MIXED * 2 + [(9, 4)] * pad, seed=18), 1)
    finally:
        for b in variants:
            ctx.set_variant(b, -1)


def test_a_captured_call_forks_and_joins(ctx):  # noqa: F811
    """A call on two streams inside a caller's graph, replayed three times
    with eager calls between."""
    import torch
    from paper_2407_19151_amd import runner
    wl = custom_workload([(9, 4)] * 400 + MIXED[:5] * 2, seed=19)
    dw, de, other = (runner.DeviceWorkload(wl) for _ in range(3))
    start = [x.clone() for x in (dw.vx, dw.vy, dw.vz)]
    runner.collide_sorted(ctx, de, 1)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        runner.collide_sorted(ctx, dw, 1, with_stats=False)
    for _ in range(3):
        runner.collide_sorted(ctx, other, 1)
        for x, x0 in zip((dw.vx, dw.vy, dw.vz), start):
            x.copy_(x0)
        g.replay()
        torch.cuda.synchronize()
        assert np.array_equal(dw.velocities(), de.velocities())
    assert ctx.device_error() == 0

"""Calls on either side of the rule that puts the 2048 and 4096 buckets alone on
the side stream (many cells with their mean in the 1024 or the 128 bucket): the
bits of a plan of the same cells, steps back to back, cells of other buckets
among them."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from gpu_helpers import custom_workload
from test_gpu_parity import ctx  # noqa: F401

OTHERS = [(40, 30), (100, 90), (200, 150), (400, 300), (700, 600), (1500, 900)]


@pytest.mark.parametrize("cell,per_cu", [((350, 350), 8), ((3, 2), 160)])
@pytest.mark.parametrize("more", [-10, 1])
@pytest.mark.parametrize("precision", [0, 1])
def test_call_and_plan_give_the_same_bits(ctx, cell, per_cu, more, precision):  # noqa: F811
    import torch
    from paper_2407_19151_amd import runner
    cu = torch.cuda.get_device_properties(0).multi_processor_count
    wl = custom_workload(OTHERS + [cell] * (per_cu * cu + more - len(OTHERS)), seed=31)
    p = runner.params_for(wl, precision=precision)
    dw, dp = runner.DeviceWorkload(wl), runner.DeviceWorkload(wl)
    plan = runner.make_plan(ctx, dp, params=p, autotune=False)
    for step in range(4):
        runner.collide_sorted(ctx, dw, step, params=p)
    plan.run(0, 4)
    assert ctx.device_error() == 0
    assert np.array_equal(dp.velocities(), dw.velocities())
    assert not np.array_equal(dw.velocities(), wl.velocities())
    plan.close()

"""The descending-weight order of species whose ties crowd the sort's buckets:
decided once per cell, ordered by value afterwards.  Two weight classes, forty
values within a few ulp of each other (past the per-value rounds), and sizes
around the bucket limit of 48, called per step and through a plan."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from gpu_helpers import check_parity, custom_workload, oracle_step
from test_gpu_parity import ctx  # noqa: F401

SIZES = [(60, 40), (70, 69), (130, 200), (700, 320), (1500, 900), (3000, 40), (5200, 6)]


@pytest.mark.parametrize("relativistic", [False, True])
@pytest.mark.parametrize("weights", ["two", "clustered"])
@pytest.mark.parametrize("many", [False, True])
def test_crowded_ties(ctx, many, weights, relativistic):  # noqa: F811
    from paper_2407_19151_amd import runner
    sizes = SIZES + [(9, 6)] * (300 if many else 0)
    wl = custom_workload(sizes, seed=91, weight_mode=weights,
                         masses=(1.0, 1836.0) if relativistic else (1.0, 100.0),
                         relativistic=relativistic, c=1.0 if relativistic else float("inf"))
    v0 = wl.velocities()
    ref = wl.copy()
    oracle_step(ref, 3)

    def rerun(p):
        oracle_step(p, 3)
        return p.velocities()

    dw, dp = runner.DeviceWorkload(wl), runner.DeviceWorkload(wl)
    runner.collide_sorted(ctx, dw, 3, with_stats=False)
    plan = runner.make_plan(ctx, dp, autotune=False)
    plan.run(3, 1)
    for d in (dw, dp):
        check_parity(wl, d.velocities(), ref.velocities(), v0, rerun=rerun)
    assert np.array_equal(dw.velocities(), dp.velocities())
    assert ctx.device_error() == 0
    plan.close()

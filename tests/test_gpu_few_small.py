"""A plan of few cells takes one wave per cell where none of the smallest bucket
holds more than 64 particles, a call of the same cells four waves: the same
bits, in every form, at sizes up to and past the wave."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from gpu_helpers import custom_workload
from test_gpu_parity import ctx  # noqa: F401

SMALL = [(i, j) for i, j in ((1, 0), (0, 2), (3, 0), (1, 1), (2, 3), (7, 4), (16, 16), (31, 30),
                             (32, 31), (33, 31), (60, 1), (1, 63), (64, 0), (32, 32))]
FORMS = [dict(precision=q, method=m, pairing=g) for q, m, g in
         ((0, 1, 0), (1, 1, 0), (0, 0, 0), (1, 0, 0), (0, 1, 1), (1, 1, 1), (0, 1, 2), (1, 1, 2))]
FORMS += [dict(max_passes=3, f_E=0.01), dict(on_failure=1, f_E=1e-4), dict(moment_correction=0),
          dict(sort_by_weight=0), dict(relativistic=1), dict(relativistic=1, pairing=1),
          dict(diagnostics=1)]


@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("more", [[], [(33, 32)], [(100, 90), (300, 250)]])
def test_plan_and_call_give_the_same_bits(ctx, form, more):  # noqa: F811
    from paper_2407_19151_amd import native, runner
    rel = "relativistic" in form
    kw = dict(masses=(1.0, 1836.0), relativistic=True, c=1.0, dt=0.003) if rel else {}
    wl = custom_workload(SMALL * 3 + more, seed=51, weight_mode="lognormal", **kw)
    p = runner.params_for(wl, **form)
    dw, dp = runner.DeviceWorkload(wl), runner.DeviceWorkload(wl)
    plan = runner.make_plan(ctx, dp, params=p, autotune=False, with_stats=True)
    for step in range(3):
        runner.collide_sorted(ctx, dw, step, params=p)
        plan.run(step, 1)
        assert np.array_equal(dp.velocities(), dw.velocities())
        assert native.read_stats(dp.stats) == native.read_stats(dw.stats)
    assert ctx.device_error() == 0
    assert not np.array_equal(dw.velocities(), wl.velocities())
    plan.close()

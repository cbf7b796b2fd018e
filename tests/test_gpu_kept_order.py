"""Cells of 1025-4096 particles without a plan: the weight order kept for the
call gives the bits of the order sorted in every collision (the allocation-free
entry, a captured call) and of a plan's, also when the context's room grows or
held another call's."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from gpu_helpers import custom_workload
from test_gpu_parity import ctx  # noqa: F401

SIZES = [(513, 512), (1024, 1), (1000, 1048), (1025, 1024), (2049, 2047), (1, 4095), (60, 50)]


@pytest.mark.parametrize("pad", [0, 300])
@pytest.mark.parametrize("weights", ["lognormal", "mixed", "two", "clustered"])
@pytest.mark.parametrize("form", ["fp64", "fp32", "relativistic"])
def test_kept_order_gives_the_same_bits(ctx, form, weights, pad):  # noqa: F811
    from paper_2407_19151_amd import runner
    over = dict(precision=1) if form == "fp32" else {}
    rel = dict(relativistic=True, c=1.0, masses=(1.0, 1836.0)) if form == "relativistic" else {}
    for sizes in (SIZES[2:3], SIZES, SIZES[3:] * 3, SIZES[::-1]):
        wl = custom_workload(sizes + [(3, 2)] * pad, seed=23, weight_mode=weights, **rel)
        p = runner.params_for(wl, **over)
        dw, dp, dn = (runner.DeviceWorkload(wl) for _ in range(3))
        runner.collide_sorted(ctx, dw, 1, params=p)
        plan = runner.make_plan(ctx, dp, params=p, autotune=False)
        plan.run(1, 1)
        plan.close()
        assert np.array_equal(dw.velocities(), dp.velocities())
        if not rel:
            ctx.collide_sorted_noalloc(
                dn.offsets, dn.w, dn.vx, dn.vy, dn.vz, n_cells=wl.n_cells, mass=wl.mass,
                charge=wl.charge, collisions=wl.collisions, dt=wl.dt, coulomb_log=wl.coulomb_log,
                seed=wl.seed, step=1, params=p, cell_volume=wl.cell_volume)
            assert np.array_equal(dw.velocities(), dn.velocities())
        assert ctx.device_error() == 0


def test_a_captured_call_holds_no_room_that_may_move(ctx):  # noqa: F811
    """Captured, then a larger call, then replayed: the eager bits."""
    import torch
    from paper_2407_19151_amd import runner
    wl = custom_workload([(1000, 1048)] * 2, seed=29, weight_mode="lognormal")
    big = custom_workload([(1000, 1048)] * 40, seed=30, weight_mode="lognormal")
    dw, de, db = runner.DeviceWorkload(wl), runner.DeviceWorkload(wl), runner.DeviceWorkload(big)
    runner.collide_sorted(ctx, db, 1)  # (the cell lists of the larger call: not what moves)
    start = [x.clone() for x in (dw.vx, dw.vy, dw.vz)]
    g = torch.cuda.CUDAGraph()
    runner.collide_sorted(ctx, de, 1)
    torch.cuda.synchronize()
    with torch.cuda.graph(g):
        runner.collide_sorted(ctx, dw, 1, with_stats=False)
    larger = runner.DeviceWorkload(custom_workload([(2000, 2048)] * 40, seed=31,
                                                   weight_mode="lognormal"))
    for _ in range(3):
        runner.collide_sorted(ctx, larger, 1)
        for x, x0 in zip((dw.vx, dw.vy, dw.vz), start):
            x.copy_(x0)
        g.replay()
        torch.cuda.synchronize()
        assert np.array_equal(dw.velocities(), de.velocities())
    assert ctx.device_error() == 0

"""The per-call entries' front kernels (one workgroup or the grid) and the
few-cells rule (up to as many cells as compute units: one kernel for the cells
of up to 1024 particles), at the sizes where they change over."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from gpu_helpers import check_parity, custom_workload, oracle_step


@pytest.fixture(scope="module")
def ctx():
    from paper_2407_19151_amd import native
    c = native.Context(0)
    yield c
    c.close()


def _n_cu():
    import torch
    return torch.cuda.get_device_properties(0).multi_processor_count


@pytest.mark.parametrize("extra", [-1, 0, 1])
@pytest.mark.parametrize("precision", [0, 1])
def test_few_cells_rule_matches_the_oracle_on_either_side(ctx, extra, precision):
    """One cell fewer than, as many as, and one more than the compute units,
    with cells in the 128, 256, 512, 1024 and 2048 buckets: parity, and a plan of the same cells gives the same bits."""
    from paper_2407_19151_amd import native, runner
    sizes = [(7, 4)] * (_n_cu() + extra - 4) + [(100, 60), (200, 170), (400, 300), (700, 500)]
    wl = custom_workload(sizes, seed=31 + extra)
    p = runner.params_for(wl, precision=precision)
    dw, dp = runner.DeviceWorkload(wl), runner.DeviceWorkload(wl)
    dw.stats.fill_(255)  # (cleared by the call)
    runner.collide_sorted(ctx, dw, 2, params=p)
    st = native.read_stats(dw.stats)
    assert ctx.device_error() == 0
    ref = wl.copy()
    so = oracle_step(ref, 2, uniform23=bool(precision))
    assert st["pairs"] == so["pairs"] and st["collisions"] == so["collisions"]
    v0 = wl.velocities()
    if precision:  # the FP32 form's bar
        scale = np.sqrt((v0 * v0).sum(0)).max()
        assert np.abs(dw.velocities() - ref.velocities()).max() <= 1e-4 * scale
    else:
        # (no comparison of the correction-pair counts: the electrons' weights
        # are equal, so their energy violation is rounding noise, 1e-17 of the
        # cell's energy, and whether it is exactly zero is the summation order's)
        check_parity(wl, dw.velocities(), ref.velocities(), v0)
    plan = runner.make_plan(ctx, dp, params=p, autotune=False)
    plan.run(2, 1)
    assert np.array_equal(dp.velocities(), dw.velocities())
    plan.close()


@pytest.mark.parametrize("sizes", [[(64, 64)] * 128, [(64, 64)] * 127 + [(65, 64)],
                                   [(1, 0)] * 16384, [(1, 0)] * 16385])
def test_front_checks_the_last_weight_and_lists_every_cell(ctx, sizes):
    """16 384 particles or cells (the most one workgroup takes) and one more:
    every cell is stepped, the last weight is checked, and the counters are
    cleared by the next call."""
    from paper_2407_19151_amd import native, runner
    wl = custom_workload(sizes, seed=7)
    dw = runner.DeviceWorkload(wl)
    for step in (0, 1):
        runner.collide_sorted(ctx, dw, step)
    assert ctx.device_error() == 0
    ref = wl.copy()
    oracle_step(ref, 0)
    so = oracle_step(ref, 1)
    st = native.read_stats(dw.stats)
    assert (st["pairs"], st["collisions"]) == (so["pairs"], so["collisions"])
    check_parity(wl, dw.velocities(), ref.velocities(), wl.velocities())
    dw.w[-1] = float("nan")
    runner.collide_sorted(ctx, dw, 2)
    assert ctx.device_error() == 4

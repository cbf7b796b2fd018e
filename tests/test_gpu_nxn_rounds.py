"""N x N rounds that hold both species' intra pairs (a dual pass), and the
duplicity form's: cells at which the rounds of both just fit a wave or a
workgroup, one particle past it, and lists of very different lengths.  Strict
parity at a step small enough to keep the chains of pairs well conditioned,
as the N x N tests do: 1e-12 sqrt(n)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from gpu_helpers import custom_workload, oracle_step, rel_err
from paper_2407_19151_amd import workloads as W
from test_gpu_parity import ctx  # noqa: F401

SIZES = [(64, 64), (64, 63), (65, 63), (66, 63), (127, 1), (128, 128), (130, 126), (3, 60),
         (2, 2), (60, 3), (256, 256), (257, 255), (258, 300), (1, 40), (40, 0)]


@pytest.mark.parametrize("over", [dict(pairing=1), dict(pairing=1, precision=1),
                                  dict(pairing=1, relativistic=1), dict(pairing=2)])
@pytest.mark.parametrize("many", [False, True])
def test_rounds_of_both_species(ctx, many, over):  # noqa: F811
    from paper_2407_19151_amd import native, runner
    rel = bool(over.get("relativistic"))
    over = {k: v for k, v in over.items() if k != "relativistic"}
    sizes = SIZES + [(9, 6)] * (300 if many else 0)
    wl = custom_workload(sizes, seed=77, weight_mode="lognormal", dt=0.05e-4 * W.tau_e(2.0),
                         masses=(1.0, 1836.0) if rel else (1.0, 100.0), relativistic=rel,
                         c=1.0 if rel else float("inf"))
    dw = runner.DeviceWorkload(wl)
    runner.collide_sorted(ctx, dw, 4, params=runner.params_for(wl, **over))
    assert ctx.device_error() == 0
    st = native.read_stats(dw.stats)
    ref = wl.copy()
    so = oracle_step(ref, 4, pairing=over["pairing"], uniform23=bool(over.get("precision")))
    assert (st["pairs"], st["collisions"]) == (so["pairs"], so["collisions"])
    err = rel_err(wl, dw.velocities(), ref.velocities(), wl.velocities())
    n = np.diff(wl.offsets).max()
    # the FP32 form: a few operations of 6e-8 per pair on changes of the small step
    assert err.max() <= (1e-4 if over.get("precision") else 1e-12 * np.sqrt(n))

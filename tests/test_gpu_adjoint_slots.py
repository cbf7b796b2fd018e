"""The reverse-mode kernels at the edges of their capacities and of their
record slots: <g, J t> of the forward mode equals <J^T g, t> per cell, cells
of one size per kernel (LDS up to 1024 particles, global scratch above),
odd and even lists, and collision lists longer than the slots (six in LDS,
three in global scratch), which the sweep takes in groups."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from gpu_helpers import custom_workload
from test_gpu_adjoint import _gpu_jvp, _gpu_vjp, _percell, _scale, ctx  # noqa: F401

LONG = [(0, 0), (1, 1), (0, 1), (1, 1), (0, 1), (0, 0), (0, 1)]
EDGES = [(64, 64), (65, 64), (128, 128), (129, 128), (256, 256), (257, 256), (512, 512),
         (513, 512), (2049, 2048)]


def _transpose(ctx, wl, bar, step=1, **pover):
    rng = np.random.default_rng(5)
    v0 = wl.velocities()
    sc = _scale(wl, v0)
    g = rng.normal(size=v0.shape) / np.maximum(sc, 1e-300)
    t = rng.normal(size=v0.shape) * sc
    jt = _gpu_jvp(ctx, wl, t, step, 0.0, **pover)
    jl = _gpu_jvp(ctx, wl, np.zeros_like(t), step, 1.0, **pover)
    gj, gl = _gpu_vjp(ctx, wl, g, step, **pover)
    left, right = _percell(wl, (g * jt).sum(0)), _percell(wl, (gj * t).sum(0))
    scale = _percell(wl, (np.abs(g * jt) + np.abs(gj * t)).sum(0))
    assert np.all(np.abs(left - right) <= bar * scale), np.max(np.abs(left - right) / scale)
    assert abs(gl - (g * jl).sum()) <= bar * np.abs(g * jl).sum()


@pytest.mark.parametrize("many", [False, True])
def test_capacities(ctx, many):  # noqa: F811
    """Every kernel at its largest cell and one particle past it; with more
    cells than compute units (the 64- and 128-thread kernels) and with few
    (256 threads).  Bar: 1e-11, as the forward and reverse modes differ in the
    association of products only."""
    sizes = EDGES + [(5, 4)] * (300 if many else 2)
    _transpose(ctx, custom_workload(sizes, seed=21), 1e-11)


@pytest.mark.parametrize("method", [0, 1])
def test_lists_longer_than_the_slots(ctx, method):  # noqa: F811
    """Seven collisions, in cells of either scratch.  Bar: 1e-10 (a product of
    seven Jacobians where the three-collision lists are held to 1e-11)."""
    wl = custom_workload([(41, 60), (300, 211), (700, 600), (2, 1)], seed=22, collisions=LONG,
                         weight_mode="lognormal", method=method)
    _transpose(ctx, wl, 1e-10)

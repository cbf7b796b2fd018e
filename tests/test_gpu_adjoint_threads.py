"""The reverse-mode kernels of cells of 1025 to 2048 particles (eight waves in
LDS; four with the caller's variant), and the caller's wide variants for
smaller cells: the transpose test of each (bar 1e-11, as for the other
kernels), and the FP32 form against its one-wave kernel, one collision from
the same state, where the two differ by the order of the per-cell sums (a few
1e-16 of the cell's scale, which the cut pair's quotient may amplify: 1e-9)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from gpu_helpers import custom_workload
from test_gpu_adjoint import _gpu_vjp, _scale, ctx  # noqa: F401
from test_gpu_adjoint_slots import LONG, _transpose

CELLS = [(513, 512), (900, 601), (1024, 1024), (2048, 0), (1, 1500)]


@pytest.mark.parametrize("variants", [{}, {4: 11}, {4: 8}, {3: 6, 2: 7, 4: 7}])
@pytest.mark.parametrize("pad", [0, 300])
def test_transpose(ctx, variants, pad):  # noqa: F811
    for b, v in variants.items():
        ctx.set_variant(b, v)
    try:
        wl = custom_workload(CELLS + [(300, 150), (500, 411)] + [(5, 4)] * pad, seed=24,
                             weight_mode="lognormal")
        _transpose(ctx, wl, 1e-11)
        if not variants:
            wl.collisions = LONG
            _transpose(ctx, wl, 1e-10)
            _transpose(ctx, wl, 1e-10, moment_correction=0)
    finally:
        for b in variants:
            ctx.set_variant(b, -1)


@pytest.mark.parametrize("variant", [-1, 11])
def test_fp32_form(ctx, variant):  # noqa: F811
    wl = custom_workload(CELLS, seed=25, weight_mode="lognormal", collisions=[(0, 1)])
    g = np.random.default_rng(6).normal(size=(3, wl.n))
    try:
        ctx.set_variant(4, variant)
        a, la = _gpu_vjp(ctx, wl, g, 2, precision=1)
        ctx.set_variant(4, 10)
        b, lb = _gpu_vjp(ctx, wl, g, 2, precision=1)
    finally:
        ctx.set_variant(4, -1)
    assert np.abs(a - g).max() > 0.1
    assert np.all(np.abs(a - b).max(0) <= 1e-9 * _scale(wl, b))
    assert abs(la - lb) <= 1e-9 * np.abs(g).sum()

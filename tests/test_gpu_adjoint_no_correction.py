"""The reverse mode without the moment correction, in every kernel: one to
four waves per cell, with more cells than compute units and with few; one
collision, three, and a list longer than the record slots.  Each follows a call
with the correction on in which every collision is reset, whose records (a
set failure flag in the same LDS words) must not be read.  Bar of the transpose
test for three collisions, 1e-11; 1e-10 for seven."""
import pytest

pytestmark = pytest.mark.gpu

from gpu_helpers import custom_workload
from test_gpu_adjoint import _gpu_vjp, ctx  # noqa: F401
from test_gpu_adjoint_slots import LONG, _transpose

CELLS = [(50, 40), (128, 120), (129, 128), (200, 256), (257, 256), (512, 500), (513, 512)]


@pytest.mark.parametrize("many", [False, True])
@pytest.mark.parametrize("coll,bar", [([(0, 0)], 1e-11), ([(0, 1)], 1e-11),
                                      ([(0, 0), (1, 1), (0, 1)], 1e-11), (LONG, 1e-10)])
def test_no_correction(ctx, many, coll, bar):  # noqa: F811
    wl = custom_workload(CELLS + [(5, 4)] * (300 if many else 2), seed=23, collisions=coll,
                         weight_mode="lognormal")
    _gpu_vjp(ctx, wl, wl.velocities(), 1, f_E=1e-9)
    _transpose(ctx, wl, bar, moment_correction=0)

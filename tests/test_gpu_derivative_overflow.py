"""The derivatives of a pair whose path length s ~ 1/|u|^3 overflows: the angle
no longer depends on s there, so the pair's Jacobian is that of a fixed
rotation, whatever the scale of u.  TA77: the full reversal, which for equal
masses and weights exchanges the two particles' tangents.  N97: the isotropic
angle, compared with the same pair at a relative speed 1e-30, whose s is finite
and as far past that limit.  Bar 1e-12: a few dozen roundings on operands that
differ by a power of ten."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from gpu_helpers import custom_workload
from test_gpu_adjoint import _gpu_jvp, _gpu_vjp, ctx  # noqa: F401


@pytest.mark.parametrize("method", [0, 1])
@pytest.mark.parametrize("mode", ["tangent", "adjoint"])
def test_pair_with_overflowing_path_length(ctx, method, mode):  # noqa: F811
    def derivative(speed):
        wl = custom_workload([(2, 0)] * 8, seed=3, method=method, collisions=[(0, 0)])
        wl.vx, wl.vy, wl.vz = speed * wl.velocities()
        x = np.random.default_rng(4).normal(size=(3, wl.n))
        if mode == "tangent":
            return x, _gpu_jvp(ctx, wl, x, 1, 0.3, moment_correction=0)
        g, gl = _gpu_vjp(ctx, wl, x, 1, moment_correction=0)
        assert abs(gl) <= 1e-12
        return x, g

    x, got = derivative(1e-120)
    want = x.reshape(3, 8, 2)[:, :, ::-1].reshape(3, 16) if method == 0 else derivative(1e-30)[1]
    assert np.abs(want - x).max() > 0.1
    assert np.abs(got - want).max() <= 1e-12 * np.abs(want).max()

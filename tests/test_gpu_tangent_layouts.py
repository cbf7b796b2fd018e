"""The differentiated form at the edges of its kernels' capacities (LDS up to
2048 particles, global scratch above), on either side of the few-cells rule,
and where the correction fails and the snapshots are restored.  Same reference
and bar as test_gpu_tangent: central differences of the oracle, 1e-6 of the
tangent's scale plus ten times the difference's own error."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from gpu_helpers import custom_workload
from test_gpu_tangent import _oracle_fd, _scale, ctx  # noqa: F401

EDGES = [(64, 64), (65, 64), (128, 128), (129, 128), (256, 256), (257, 256), (512, 512),
         (513, 512), (1024, 1024), (1025, 1024), (2, 1), (1, 0), (0, 2)]


@pytest.mark.parametrize("pad", [0, 300])
@pytest.mark.parametrize("f_E", [0.05, 0.002])
@pytest.mark.parametrize("weights", ["mixed", "two"])
def test_tangent_at_capacity_edges(ctx, pad, f_E, weights):  # noqa: F811
    import torch
    from paper_2407_19151_amd import runner
    wl = custom_workload(EDGES + [(3, 2)] * pad, seed=91, weight_mode=weights)
    wl.f_E = f_E
    v0 = wl.velocities().copy()
    t = np.random.default_rng(3).normal(size=v0.shape) * _scale(wl, v0)
    dw = runner.DeviceWorkload(wl)
    T = torch.as_tensor(t, device="cuda").contiguous()
    runner.collide_sorted_jvp(ctx, dw, T, 2, coulomb_log_tangent=0.5)
    assert ctx.device_error() == 0
    jt = T.cpu().numpy()
    fd1, flip1 = _oracle_fd(wl, t, 2, 0.5, 1e-6)
    fd2, flip2 = _oracle_fd(wl, t, 2, 0.5, 5e-7)
    keep = ~(flip1 | flip2)[wl.cells]
    sc = np.maximum(_scale(wl, fd2), 1e-300)
    err = np.abs(jt - fd2).max(0) / sc
    est = np.abs(fd1 - fd2).max(0) / sc
    assert keep.mean() > 0.5 and np.all(np.isfinite(jt))
    assert np.all(err[keep] <= 1e-6 + 10.0 * est[keep])

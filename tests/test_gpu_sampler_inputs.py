"""The angle sampler alone at path lengths that no pair has (zero, negative,
infinities, NaN): no deflection where s is not positive, the isotropic angle
at infinity, in every form."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from test_gpu_parity import ctx  # noqa: F401


@pytest.mark.parametrize("precision", [0, 1])
def test_n97_path_lengths_out_of_range(ctx, precision):  # noqa: F811
    import torch
    s = np.array([0.0, -0.0, -1e-300, -0.5, -3.0, -40.0, -1e30, -np.inf, np.nan, np.inf])
    a0 = np.full(s.size, 0x30000000, dtype=np.int32)
    oc, st, A = (x.cpu().numpy() for x in ctx.sample_angles(
        1, precision, torch.from_numpy(s).cuda(), torch.from_numpy(a0).cuda(),
        torch.from_numpy(a0).cuda()))
    assert np.all(oc[:-1] == 0.0) and np.all(st[:-1] == 0.0) and np.all(np.isinf(A[:-1]))
    assert A[-1] == 0.0 and abs(oc[-1] - 0.375) < 1e-6

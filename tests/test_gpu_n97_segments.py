"""The FP64 N97 sampler at the edges of its segments (powers of two, the
switch of representation at s = 2, the series from 8, the isotropic limit from
50) against the oracle.  Uniforms up to 0.9, where 1 - cos theta is at most
five times more sensitive than its operands: a handful of roundings on either
side, so 5e-15 relative."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import oracle
from paper_2407_19151_amd import workloads as W
from test_gpu_parity import ctx  # noqa: F401


def test_segment_edges(ctx):  # noqa: F811
    import torch
    edges = [2.0 ** -6 * (1.0 + k / 32.0) * 2.0 ** e for e in range(-1, 9) for k in range(32)]
    edges += [8.0, 20.0, 36.5, 50.0, 64.0, 700.0, 1e-300, 2.0 ** -40]
    s = np.array([f(x) for x in edges for f in (lambda x: x, lambda x: np.nextafter(x, 0.0),
                                                lambda x: np.nextafter(x, 1e9))])
    s = np.repeat(s, 4)
    rng = np.random.default_rng(3)
    a0 = (rng.uniform(1e-6, 0.9, s.size) * 2.0 ** 32).astype(np.uint32)
    a1 = np.zeros_like(a0)
    oc, st, A = (x.cpu().numpy() for x in ctx.sample_angles(
        W.N97, 0, torch.from_numpy(s).cuda(), torch.from_numpy(a0.view(np.int32)).cuda(),
        torch.from_numpy(a1.view(np.int32)).cuda()))
    for i in range(s.size):
        ro, _ = oracle.sample_angle(W.N97, float(s[i]), (float(a0[i]) + 0.5) * 2.0 ** -32, 0.5)
        ra = oracle.n97_A(float(s[i]))
        assert abs(oc[i] - ro) <= 5e-15 * ro, (s[i], a0[i], oc[i], ro)
        assert abs(A[i] - ra) <= 5e-15 * ra, (s[i], A[i], ra)

"""The unsorted entry on either side of 2^24 particles with three radix passes
(records below, the payload moved with the keys from there): the same bits as
a stable sort, the sorted step and a scatter back."""
import pytest

pytestmark = pytest.mark.gpu

from test_gpu_parity import ctx  # noqa: F401
from test_gpu_unsorted_passes import ARGS


@pytest.mark.parametrize("n", [(1 << 24) - 1, 1 << 24])
def test_three_passes(ctx, n):  # noqa: F811
    import torch
    n_cells = 200_003
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    key = torch.randint(0, 2 * n_cells, (n,), generator=g, device="cuda")
    w = torch.rand(n, generator=g, device="cuda", dtype=torch.float64) + 1.0
    v = torch.randn((3, n), generator=g, device="cuda", dtype=torch.float64)
    skey, perm = torch.sort(key, stable=True)
    off = torch.searchsorted(skey, torch.arange(2 * n_cells + 1, device="cuda"))
    gw, gv = w[perm].contiguous(), v[:, perm].contiguous()
    ctx.collide_sorted(off, gw, *gv, n_cells=n_cells, step=4, **ARGS)
    want = torch.empty_like(v)
    want[:, perm] = gv
    got = v.clone()
    ctx.collide((key // 2).to(torch.int32), (key % 2).to(torch.int32), w, *got, n_cells=n_cells,
                step=4, **ARGS)
    assert ctx.device_error() == 0
    assert torch.equal(got, want) and not torch.equal(got, v)

"""The unsorted entry's way there and back (one radix pass up to 511 groups,
two up to 2^18 - 1, three up to 2^27 - 1, four above; tiles of 4096 particles)
against a stable sort, the sorted step and a scatter back: the same bits."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from test_gpu_parity import ctx  # noqa: F401

ARGS = dict(mass=[1.0, 1.0], charge=[-1.0, 2.0], collisions=[(0, 0), (0, 1), (1, 1)], dt=0.05,
            coulomb_log=8.0, seed=77)


@pytest.mark.parametrize("n_cells,sizes", [
    (3, [1, 2, 4095, 4096, 4097]),
    (255, [0, 4096, 8 * 4096 - 1, 40000]),
    (256, [4097, 8 * 4096 + 1]),
    (5003, [3, 9 * 4096, 100003]),
    (131072, [4095, 300001]),
    (1 << 26, [60001]),
])
@pytest.mark.parametrize("invalid", [False, True])
def test_unsorted_step_is_the_sorted_one_in_another_order(ctx, n_cells, sizes, invalid):  # noqa: F811
    import torch
    rng = np.random.default_rng(n_cells)
    for n in sizes:
        # (a few cells of the whole range hold the particles, so that they meet)
        pool = np.unique(np.concatenate([[0, n_cells - 1],
                                         rng.integers(0, n_cells, max(1, n // 50))]))
        cells = rng.choice(pool, n).astype(np.int32)
        sp = rng.integers(0, 2, n).astype(np.int32)
        if invalid:
            cells[rng.integers(0, n, n // 40)] = n_cells
            sp[rng.integers(0, n, n // 40)] = -1
        bad = (cells >= n_cells) | (sp < 0)
        key = np.where(bad, 2 * n_cells, cells.astype(np.int64) * 2 + sp)
        perm = torch.from_numpy(np.argsort(key, kind="stable")).cuda()
        w = torch.from_numpy(rng.uniform(1.0, 3.0, n)).cuda()
        v = torch.from_numpy(rng.normal(size=(3, n))).cuda()
        key = torch.from_numpy(np.sort(key)).cuda()
        off = torch.searchsorted(key, torch.arange(2 * n_cells + 1, device="cuda"))
        gw, gv = w[perm].contiguous(), v[:, perm].contiguous()
        ctx.collide_sorted(off, gw, *gv, n_cells=n_cells, step=4, **ARGS)
        assert ctx.device_error() == 0
        want = torch.empty_like(v)
        want[:, perm] = gv
        got, w0 = v.clone(), w.clone()
        ctx.collide(torch.from_numpy(cells).cuda(), torch.from_numpy(sp).cuda(), w, *got,
                    n_cells=n_cells, step=4, **ARGS)
        assert ctx.device_error() == (3 if bad.any() else 0)
        assert torch.equal(got, want) and torch.equal(w, w0), n
        moved = (got != v).any(0).cpu().numpy()
        assert not moved[bad].any()
        if n > 100:
            assert moved[~bad].mean() > 0.5

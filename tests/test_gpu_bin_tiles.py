"""Binning at the edges of its tiles (4096 items), of the tile ranges of the
eight XCDs and of its passes (9 bits of the group key each), bit for bit
against numpy's stable sort."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from test_gpu_parity import ctx  # noqa: F401

SIZES = [1, 63, 64, 65, 1023, 4095, 4096, 4097, 8 * 4096 - 1, 8 * 4096, 8 * 4096 + 1,
         17 * 4096 + 5, 200003]


@pytest.mark.parametrize("n_cells,S", [(1, 1), (511, 1), (512, 1), (170, 3), (87382, 3),
                                       (134217, 2)])
@pytest.mark.parametrize("order", ["random", "sorted", "one group", "some invalid"])
def test_bin_edges(ctx, n_cells, S, order):  # noqa: F811
    import torch
    rng = np.random.default_rng(n_cells + S)
    for n in SIZES:
        cells = rng.integers(0, n_cells, n).astype(np.int32)
        sp = rng.integers(0, S, n).astype(np.int32)
        if order == "sorted":
            cells.sort()
        if order == "one group":
            cells[:], sp[:] = n_cells - 1, S - 1
        if order == "some invalid":
            cells[rng.integers(0, n, max(1, n // 50))] = -1
            sp[rng.integers(0, n, max(1, n // 50))] = S
        bad = (cells < 0) | (sp < 0) | (sp >= S)
        key = np.where(bad, n_cells * S, cells.astype(np.int64) * S + sp)
        off, perm = ctx.bin(torch.from_numpy(cells).cuda(), torch.from_numpy(sp).cuda(), n_cells,
                            S)
        assert np.array_equal(perm.cpu().numpy(), np.argsort(key, kind="stable")), n
        want = np.searchsorted(np.sort(key), np.arange(n_cells * S + 1))
        assert np.array_equal(off.cpu().numpy(), want), n
        assert ctx.device_error() == (3 if bad.any() else 0)

"""The relativistic kernels in the compact layout, in the cells that used to
take another one (2049-4096 particles, and every size for the diagnostic and
duplicity forms), and the correction walking over several groups of 64 pairs."""
import pytest

pytestmark = pytest.mark.gpu

from gpu_helpers import custom_workload
from test_gpu_parity import _parity, ctx  # noqa: F401


def _cells(sizes, seed, weights="lognormal"):
    return custom_workload(sizes, seed=seed, masses=(1.0, 1836.0), relativistic=True, c=1.0,
                           weight_mode=weights)


@pytest.mark.parametrize("over", [{}, {"diagnostics": 1}, {"pairing": 2}])
@pytest.mark.parametrize("sizes", [[(64, 64), (129, 127), (257, 255), (513, 511)],
                                   [(1025, 1023), (2000, 2096)]])
def test_compact_layout_parity(ctx, sizes, over):  # noqa: F811
    """Cells that fill each capacity, odd and even lists."""
    _parity(ctx, _cells(sizes, 61), 1, **over)


@pytest.mark.parametrize("f_E", [0.05, 0.002])
def test_correction_past_the_first_64_pairs(ctx, f_E):  # noqa: F811
    """A small f_E spreads the correction over hundreds of pairs and makes it
    fail in some cells (reset there)."""
    wl = _cells([(300, 200), (41, 500), (900, 90), (7, 3), (130, 2)], 62)
    _, sg, so = _parity(ctx, wl, 2, f_E=f_E)
    if f_E < 0.01:
        assert so["corr_pairs"] > 64 * len(wl.collisions)

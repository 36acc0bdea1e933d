"""Moments of small cells beside large ones, which have a launch of their own:
capacities around the limit of 2,048 slots (a cell of n has 5 n / 4 + 32)."""
import pytest

import test_gpu_moments_shapes as shapes

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hc():
    from paper_2606_31548_amd import hcao
    hcao.load_library()
    return hcao


@pytest.mark.parametrize("extra", [0, 11])
@pytest.mark.parametrize("sizes", [(1612, 1613, 1614, 63, 0, 5) + (16,) * 8, (20, 30, 1, 4097, 9001, 1281) + (40,) * 9])
def test_large_cells_among_small_ones(orc, hc, extra, sizes):
    shapes.test_moments_per_cell_match(orc, hc, extra, sizes)

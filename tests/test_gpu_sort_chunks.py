"""Loads whose cell count or particle count sits at the edges of the prefix
sums' chunks (4,096 entries) and of the radix sort's tiles: particles come back
in the stable order by cell."""
import numpy as np
import pytest

from paper_2606_31548_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cells", [1, 255, 4095, 4096, 4097, 70001])
@pytest.mark.parametrize("n", [1, 4096, 4097, 65537])
def test_load_keeps_the_stable_order(cells, n):
    from paper_2606_31548_amd import hcao
    wl = W.methane_argon(n_cells=cells, per_cell=4)
    wl.capacity_per_cell = n if cells == 1 else 0
    g = hcao.from_workload(wl)
    rng = np.random.default_rng([cells, n])
    cell = rng.integers(0, cells, n).astype(np.uint32)
    sp = rng.integers(1, 2, n).astype(np.uint8)
    vel = rng.standard_normal((n, 3)) * 500.0
    lv = np.zeros((n, 9), np.uint16)
    g.load_particles(cell, sp, vel, lv)
    order = np.argsort(cell, kind="stable")
    c, s, v, _ = g.read_particles()
    assert np.array_equal(c, np.bincount(cell, minlength=cells))
    assert np.array_equal(s, sp[order]) and np.array_equal(v, vel[order])

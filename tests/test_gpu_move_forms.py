"""The move pass with one wave per cell, with a workgroup's four waves for its
large cells, and with four waves per cell throughout: cells around the lengths
of a chunk, bitwise against the oracle."""
import numpy as np
import pytest

from paper_2606_31548_amd import workloads as W
from test_gpu_parity import _compare_state

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hc():
    from paper_2606_31548_amd import hcao
    hcao.load_library()
    return hcao


def _box(grid, per_cell, sizes, faces):
    wl = W.spatial_box(*grid, per_cell=per_cell, t_trans=20000.0, dt=5e-10, seed=9,
                       periodic=0b110 if faces else 0b111, open_faces=faces)
    wl.counts = wl.counts.copy()
    for at, n in sizes.items():
        wl.counts[at] = [n // 10, n - n // 10, 0, 0, 0]
    wl.capacity_per_cell = 0
    return wl


# at least 4,096 small cells: a wave per cell (chunks of 128), four waves above 1,024 particles (chunks of 256);
# fewer: four waves per cell; no cell above 1,024 slots: a wave per cell without the test for it
_MANY = ((16, 16, 17), 24, {0: 0, 3: 127, 9: 128, 13: 129, 1000: 1024, 1001: 1025, 2003: 1281, 4000: 3001, 4351: 1300})
_SMALL = ((16, 16, 17), 24, {0: 0, 3: 127, 9: 128, 13: 129, 1000: 257, 4351: 385})
_FEW = ((5, 4, 3), 90, {0: 0, 7: 255, 20: 256, 31: 257, 44: 513, 59: 2001})


@pytest.mark.parametrize("grid,per_cell,sizes", [_MANY, _SMALL, _FEW])
@pytest.mark.parametrize("faces", [0, 3])
def test_move_forms_parity(orc, hc, grid, per_cell, sizes, faces):
    wl = _box(grid, per_cell, sizes, faces)
    o = orc.from_workload(wl)
    g = hc.from_workload(wl)
    o.init_thermal(wl.counts, wl.t_trans, wl.t_vib)
    g.init_thermal(wl.counts, wl.t_trans, wl.t_vib)
    for n in (1, 2):
        o.step(wl.dt, n)
        g.step(wl.dt, n)
        g.sync()
        _compare_state(o, g, f"{grid} faces {faces}")
        a = np.concatenate([o.read_pos(c) for c in range(wl.n_cells)])
        assert np.array_equal(a.view(np.uint64), g.read_positions().view(np.uint64))


@pytest.mark.parametrize("grid,per_cell,sizes", [_MANY, _SMALL, _FEW])
def test_move_forms_mixed(hc, grid, per_cell, sizes):
    """The mixed form: no particle lost or doubled, each in its cell."""
    wl = _box(grid, per_cell, sizes, 0)
    g = hc.from_workload(wl, precision=hc.MIXED)
    g.init_thermal(wl.counts, wl.t_trans, wl.t_vib)
    before = g.moments()
    g.step(wl.dt, 3)
    after = g.moments()
    counts, tot = g.counts()
    births = int(g.cell_state()[2][:, hc.CTR_BIRTHS].sum())
    assert tot == before.n_total + births == after.n_total
    pos = g.read_positions()
    nx, ny, nz, lx, ly, lz, _ = wl.domain
    ijk = np.floor(pos / np.array([lx / nx, ly / ny, lz / nz])).astype(int)
    cell = ijk[:, 0] + nx * (ijk[:, 1] + ny * ijk[:, 2])
    assert np.array_equal(cell, np.repeat(np.arange(wl.n_cells), counts.astype(int)))

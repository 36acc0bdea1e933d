"""Read-back of whole states: packed on the device in bounded chunks. Uneven
cells, empty ones, one cell longer than a chunk; loads and re-loads of equal and
other sizes into one context."""
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


def _state(counts, seed):
    rng = np.random.default_rng(seed)
    n = int(np.sum(counts))
    cell = np.repeat(np.arange(len(counts), dtype=np.uint32), counts)
    sp = rng.integers(0, 5, n).astype(np.uint8)
    vel = rng.standard_normal((n, 3)).astype(np.float32).astype(np.float64) * 500.0
    lv = rng.integers(0, 4, (n, 9)).astype(np.uint16)
    lv[np.arange(9)[None, :] >= np.array([9, 0, 6, 0, 1])[sp][:, None]] = 0
    return cell, sp, vel, lv


@pytest.mark.parametrize("precision", [0, 1])
def test_load_and_read(precision):
    from paper_2606_31548_amd import hcao
    sizes = [[0, 1, 0, 257, 64, 0, 1000], [255, 0, 0, 3, 64, 1000, 0], [7, 9, 0, 0, 0, 0, 1]]
    wl = W.methane_argon(n_cells=7, per_cell=16)
    g = hcao.from_workload(wl, precision=precision)
    for seed, counts in enumerate(sizes + sizes[:1]):
        cell, sp, vel, lv = _state(counts, seed)
        kept = vel.astype(np.float32).astype(np.float64) if precision else vel  # the mixed form stores fp32
        order = np.random.default_rng(seed).permutation(len(cell))
        g.load_particles(cell[order], sp[order], vel[order], lv[order])
        back = np.argsort(cell[order], kind="stable")
        c, s, v, l = g.read_particles()
        assert np.array_equal(c, counts) and np.array_equal(s, sp[order][back])
        assert np.array_equal(v, kept[order][back]) and np.array_equal(l, lv[order][back])


def test_cell_longer_than_a_chunk():
    from paper_2606_31548_amd import hcao
    counts = [5, (4 << 20) + 77, 300]
    wl = W.methane_argon(n_cells=3, per_cell=16)
    cell, sp, vel, lv = _state(counts, 3)
    g = hcao.from_workload(wl)
    g.load_particles(cell, sp, vel, lv)
    c, s, v, l = g.read_particles()
    assert np.array_equal(c, counts) and np.array_equal(s, sp) and np.array_equal(v, vel) and np.array_equal(l, lv)


@pytest.mark.parametrize("cells,per_cell", [(13107, 8), (13108, 14), (30001, 23)])
def test_large_reads_match_the_oracle(orc, hc, cells, per_cell):
    """Counters just below and above the 4 MiB from which a read goes through
    pinned slots, and reads of more 2 MiB chunks than there are slots, the
    last one ragged."""
    wl = W.methane_argon(n_cells=cells, per_cell=per_cell, seed=5)
    o, g = orc.from_workload(wl), hc.from_workload(wl)
    o.init_thermal(wl.counts, wl.t_trans, wl.t_vib)
    g.init_thermal(wl.counts, wl.t_trans, wl.t_vib)
    for n in (1, 2):  # the second read takes the slots of the first
        o.step(wl.dt, n)
        g.step(wl.dt, n)
        g.sync()
        _compare_state(o, g, f"{cells} cells")

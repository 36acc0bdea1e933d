"""Admissions through open faces with one, four and eight lanes per molecule
(the kernel's width follows the number admitted in a step), against the fp64
oracle bit for bit: levels and rotational energies come from the same
positions of every admission's stream whichever lane draws them."""
import numpy as np
import pytest

from paper_2606_31548_amd import workloads as W
from test_gpu_parity import _compare_state
from test_gpu_spatial import _compare_pos

pytestmark = pytest.mark.gpu

EIGHT, FOUR = 16384, 196608  # the most admissions of a step that take eight and four lanes


@pytest.fixture(scope="module")
def hc():
    from paper_2606_31548_amd import hcao
    hcao.load_library()
    return hcao


@pytest.mark.parametrize("per_cell,lo,hi", [(150, 0, EIGHT), (1500, EIGHT + 1, FOUR), (14000, FOUR + 1, 10 ** 6)])
@pytest.mark.parametrize("rotors", [False, True])
def test_admissions_match_at_every_width(orc, hc, per_cell, lo, hi, rotors):
    wl = W.spatial_box(nx=5, ny=4, nz=3, per_cell=per_cell, chemistry=True, t_trans=9000.0, t_vib=4000.0, dt=1e-8,
                       open_faces=0b111111, empty=True, seed=11)
    if rotors:  # an odd number of draws before the next molecule's normals
        for s in wl.species:
            if s.n_modes:
                s.zeta_rot = 2 if s.n_modes == 1 else 3
    o, g = orc.from_workload(wl), hc.from_workload(wl)
    o.init_thermal(wl.counts, wl.t_trans, wl.t_vib)
    g.init_thermal(wl.counts, wl.t_trans, wl.t_vib)
    o.step(wl.dt, 1)
    g.step(wl.dt, 1)
    g.sync()
    admitted = g.flux_counts()[0]
    assert lo <= admitted <= hi
    assert o.flux_counts() == g.flux_counts()
    _compare_state(o, g, f"{admitted} admitted")
    _compare_pos(o, g, f"{admitted} admitted")
    if rotors:
        rot = np.concatenate([o.read_rot(c) for c in range(wl.n_cells)])
        assert np.array_equal(rot.view(np.uint64), g.read_rotational_energy().view(np.uint64))

"""Cells whose per-pair records are reduced by all waves, and products listed
in LDS or found by scanning: around the candidate threshold of a big cell and
beyond the list's length, beside small cells in the same workgroup."""
import numpy as np
import pytest

from paper_2606_31548_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hc():
    from paper_2606_31548_amd import hcao
    hcao.load_library()
    return hcao


def _uneven(sizes, t, dt):
    wl = W.methane_chemistry(n_cells=len(sizes), per_cell=64, t=t, dt=dt)
    n = np.asarray(sizes)
    wl.counts = np.stack([n // 4, 0 * n, n // 4, n // 4, n - 3 * (n // 4)], axis=1)
    wl.cell_weight = W.DENSITY * wl.cell_volume / n
    return wl


# the first steps test half of the particles, so 1,023 .. 1,027 particles lie around 512 candidates
@pytest.mark.parametrize("sizes", [[1023], [1025], [1027, 40, 3000], [33, 2050, 64, 1024, 20]])
@pytest.mark.parametrize("t,dt", [(8000.0, 5e-9), (40000.0, 2e-8)])  # the hot one: more products per step than listed
def test_parity_and_shapes(orc, hc, sizes, t, dt):
    wl = _uneven(sizes, t, dt)
    o = orc.from_workload(wl)
    o.init_thermal(wl.counts, wl.t_trans, wl.t_vib)
    o.step(wl.dt, 5)
    oc, osp, ov, ol = o.read_all()
    mixed = []
    for shape in (None, (64, 1024), (128, 8192), (512, 8192)):
        for precision in (0, 1):
            g = hc.from_workload(wl, precision=precision)
            if shape:
                g.set_launch_shape(*shape)
            g.init_thermal(wl.counts, wl.t_trans, wl.t_vib)
            g.step(wl.dt, 5)
            g.sync()
            c, s, v, l = g.read_particles()
            if precision == 0:
                assert np.array_equal(c, oc) and np.array_equal(s, osp) and np.array_equal(l, ol)
                assert np.array_equal(v.view(np.uint64), ov.view(np.uint64))
                assert np.array_equal(g.cell_state()[2], o.counters())
            else:
                mixed.append((c, s, v, l, g.cell_state()[0]))
                m = g.moments()
                assert abs(m.E_defect_J) < 1e-6 * m.E_kin_J
    for other in mixed[1:]:
        assert all(np.array_equal(a, b) for a, b in zip(mixed[0], other))

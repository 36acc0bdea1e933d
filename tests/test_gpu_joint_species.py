"""Several joint-sampled species of different mode counts in the same waves:
lanes that own a molecule of one species test trials of another. Bitwise
against the oracle in fp64, shape against shape in both forms."""
import numpy as np
import pytest

from paper_2606_31548_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hc():
    from paper_2606_31548_amd import hcao
    hcao.load_library()
    return hcao


def _chemistry():
    """Nine, six and one mode (CH4, CH3, H2), small uneven cells, reactions on."""
    wl = W.methane_chemistry(n_cells=11, per_cell=61, t=15000.0)
    for s in (W.CH4, W.CH3, W.H2):
        wl.species[s].sampler = W.SAMPLER_JOINT
    return wl


def _auto():
    """A three-mode and a four-mode triatomic, which take the joint sampler by
    default, beside a diatomic and atoms that do not."""
    wl = W.triatomic_reservoir(2003, dissociation=False, seed=5)
    wl.species.append(W.Species("D", 44 * W.AMU, bend_theta_K=[W.theta_from_wavenumber(670.0)] * 2,
                                omega_e_per_m=[1300e2, 2300e2], chi_e=[0.006] * 2, De_J=[5.5 * W.EV] * 2))
    wl.counts = np.array([[903, 100, 300, 700]])
    return wl


@pytest.mark.parametrize("make", [_chemistry, _auto])
@pytest.mark.parametrize("precision", [0, 1])
def test_mode_counts_share_a_wave(orc, hc, make, precision):
    wl = make()
    runs = []
    for shape in (None, (64, 512), (128, 2560), (256, 4096)):
        g = hc.from_workload(wl, precision=precision)
        if shape:
            g.set_launch_shape(*shape)
        g.init_thermal(wl.counts, wl.t_trans, wl.t_vib)
        g.step(wl.dt, 6)
        runs.append((*g.read_particles(), g.cell_state()[2]))
        g.close()
    for other in runs[1:]:
        assert all(np.array_equal(a, b) for a, b in zip(runs[0], other))
    if precision == 0:
        o = orc.from_workload(wl)
        o.init_thermal(wl.counts, wl.t_trans, wl.t_vib)
        o.step(wl.dt, 6)
        oc, osp, ov, ol = o.read_all()
        c, s, v, l, ctr = runs[0]
        assert np.array_equal(c, oc) and np.array_equal(s, osp) and np.array_equal(l, ol)
        assert np.array_equal(v.view(np.uint64), ov.view(np.uint64))
        assert np.array_equal(ctr, o.counters())

"""Joint sampler shared out over a wave's lanes, and the shapes the library
picks for small contexts: bitwise against the oracle."""
import numpy as np
import pytest

from paper_2606_31548_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hc():
    from paper_2606_31548_amd import hcao
    hcao.load_library()
    return hcao


def _run(hc, wl, steps, shape=None, precision=0):
    g = hc.from_workload(wl, precision=precision)
    if shape:
        g.set_launch_shape(*shape)
    g.init_thermal(wl.counts, wl.t_trans, wl.t_vib)
    g.step(wl.dt, steps)
    g.sync()
    return g


def _same(g, o):
    gc, gsp, gv, gl = g.read_particles()
    oc, osp, ov, ol = o.read_all()
    assert np.array_equal(gc, oc) and np.array_equal(gsp, osp) and np.array_equal(gl, ol)
    assert np.array_equal(gv.view(np.uint64), ov.view(np.uint64))
    assert np.array_equal(g.cell_state()[2], o.counters())


# one pair, fewer pairs than lanes, one wave's worth and its neighbours, several waves of a wide workgroup
@pytest.mark.parametrize("n", [2, 3, 66, 127, 129, 258, 1027, 5003])
def test_joint_sampler_and_default_shapes(orc, hc, n):
    wl = W.triatomic_reservoir(n, sampler=W.SAMPLER_JOINT, seed=n)
    o = orc.from_workload(wl)
    o.init_thermal(wl.counts, wl.t_trans, wl.t_vib)
    o.step(wl.dt, 6)
    for shape in (None, (64, 1024), (256, 4096)):
        _same(_run(hc, wl, 6, shape), o)


@pytest.mark.parametrize("precision", [0, 1])
def test_joint_sampler_with_mixed_samplers(orc, hc, precision):
    """Molecules of both samplers in one wave: CH3 on the joint sampler (six
    modes, many trials), CH4 and H2 on the sweep; small uneven cells."""
    wl = W.methane_chemistry(n_cells=11, per_cell=61, t=15000.0)
    wl.species[W.CH3].sampler = W.SAMPLER_JOINT
    a = _run(hc, wl, 8, None, precision)
    b = _run(hc, wl, 8, (128, 2560), precision)
    for x, y in zip(a.read_particles(), b.read_particles()):
        assert np.array_equal(x, y)
    if precision == 0:
        o = orc.from_workload(wl)
        o.init_thermal(wl.counts, wl.t_trans, wl.t_vib)
        o.step(wl.dt, 8)
        _same(a, o)

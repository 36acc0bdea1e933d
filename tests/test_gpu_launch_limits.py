"""Launch shapes at the edge of a workgroup's LDS: what a context may hold does
not depend on the joint sampler's own slots."""
import numpy as np
import pytest

from paper_2606_31548_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hc():
    from paper_2606_31548_amd import hcao
    hcao.load_library()
    return hcao


def _state(g):
    return (*g.read_particles(), *g.cell_state())


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("how", ["call", "environment"])
def test_joint_sampler_in_the_widest_workgroup(orc, hc, monkeypatch, precision, how):
    """The five-species methane chemistry (54 KB of cells, tables and levels at
    512 lanes) with a joint-sampled species besides."""
    wl = W.methane_chemistry(n_cells=5, per_cell=301, t=15000.0)
    wl.species[W.CH3].sampler = W.SAMPLER_JOINT
    runs = []
    for block in (64, 512):
        if how == "environment":
            monkeypatch.setenv("HCAO_BLOCK", str(block))
            monkeypatch.setenv("HCAO_GROUP_SLOTS", "2048")
        g = hc.from_workload(wl, precision=precision)
        if how == "call":
            g.set_launch_shape(block, 2048)
        g.init_thermal(wl.counts, wl.t_trans, wl.t_vib)
        g.step(wl.dt, 5)
        runs.append(_state(g))
        g.close()
    assert all(np.array_equal(a, b) for a, b in zip(*runs))
    if precision == 0:
        o = orc.from_workload(wl)
        o.init_thermal(wl.counts, wl.t_trans, wl.t_vib)
        o.step(wl.dt, 5)
        oc, osp, ov, ol = o.read_all()
        c, s, v, l = runs[1][:4]
        assert np.array_equal(c, oc) and np.array_equal(s, osp) and np.array_equal(l, ol)
        assert np.array_equal(v.view(np.uint64), ov.view(np.uint64))


# more groups than the chip holds at once cost a second round of them: half as much again and more
@pytest.mark.parametrize("cells,per_cell,exact", [(1536, 256, False), (2975, 256, False), (2000, 256, True),
                                                  (12000, 100, False), (1000, 560, False)])
def test_automatic_shape_fits_the_chip(hc, cells, per_cell, exact):
    """The automatic shape against 64 lanes and 1,023 slots, step time: a fifth
    of slack over the 4% (exact sampler: 8%) that the rule gives away at most."""
    wl = W.methane_chemistry(n_cells=cells, per_cell=per_cell, seed=3)
    if exact:
        for s in wl.species:
            if s.n_modes:
                s.sampler = W.SAMPLER_EXACT
    g = hc.from_workload(wl)
    best = []
    for shape in (None, (64, 1023)):
        if shape:
            g.set_launch_shape(*shape)
        g.init_thermal(wl.counts, wl.t_trans, wl.t_vib)
        g.step(wl.dt, 40)
        g.sync()
        times = []
        for _ in range(5):
            g.set_timing(True)
            g.step(wl.dt, 20)
            g.sync()
            times.append(g.kernel_time()[0])
        best.append(min(times))
    assert best[0] < 1.2 * best[1], best


def _step_ms(g, wl, steps=20):
    g.step(wl.dt, steps)
    g.sync()
    times = []
    for _ in range(5):
        g.set_timing(True)
        g.step(wl.dt, steps)
        g.sync()
        times.append(g.kernel_time()[0])
    return min(times)


def test_default_shape_can_be_read_set_and_tuned(hc):
    """One reservoir, which the default shape runs 1,024 lanes wide: setting the
    shape that was read, going back to it and tuning keep that speed (256 lanes
    take 1.7 times as long, 64 take six times)."""
    wl = W.triatomic_reservoir(10000, seed=4)
    g = hc.from_workload(wl)
    g.init_thermal(wl.counts, wl.t_trans, wl.t_vib)
    g.step(wl.dt, 20)
    first = _step_ms(g, wl)
    shape = g.launch_shape()
    assert shape == {"block": 64, "group_slots": 1024, "steps_per_launch": 0}
    g.set_launch_shape(**shape)
    assert _step_ms(g, wl) < 1.15 * first
    g.set_launch_shape(128, 2560)
    g.set_launch_shape(**shape)
    assert _step_ms(g, wl) < 1.15 * first
    tuned = g.autotune(wl.dt, trial_steps=20)
    assert _step_ms(g, wl) < 1.15 * first
    g.set_launch_shape(**tuned)
    assert _step_ms(g, wl) < 1.15 * first

"""Exact recombination sum of species without two like modes, which takes no
weights: prefixes that cover all modes and prefixes that leave modes to the
walk, against the oracle's sum."""
import numpy as np
import pytest

from paper_2606_31548_amd import workloads as W

pytestmark = pytest.mark.gpu

T = np.array([800.0, 2500.0, 6000.0, 20000.0])


def _context(thetas, stretches):
    from paper_2606_31548_amd import hcao
    we = [2300.0 * 100.0 * s for s in stretches]
    wl = W.methane_argon(n_cells=1, per_cell=16)
    wl.species = [W.Species("X", 44 * W.AMU, bend_theta_K=list(thetas), omega_e_per_m=we, chi_e=[0.012] * len(we),
                            De_J=[4.0 * W.EV] * len(we))]
    wl.reactions = []
    return hcao, wl


@pytest.mark.parametrize("thetas,stretches,de", [
    ((900.0, 1500.0), (), 1.0), ((), (1.0, 0.8), 1.5), ((1200.0, 900.0), (0.8, 1.0, 0.9), 1.2),
    ((100.0, 101.0, 102.0, 103.0), (), 0.4), ((150.0, 120.0, 110.0), (0.05, 0.06), 0.25)])
def test_distinct_modes(orc, thetas, stretches, de):
    hcao, wl = _context(thetas, stretches)
    g, o = hcao.from_workload(wl), orc.from_workload(wl)
    p, _, n = g.recombination_exact(0, de * W.EV, 0.74, T)
    want = np.array([o.rec_exact_probability(0, de * W.EV, 0.74, t) for t in T])
    # sums of positive terms in fp64 on both sides, up to 1e6 of them
    assert np.all(np.abs(p / want - 1.0) < 1e-12)
    levels = [W.K_BOLTZ * t * np.arange(4000) for t in thetas] + [g.levels(0, len(thetas) + i) - g.levels(0, len(thetas) + i)[0]
                                                                 for i in range(len(stretches))]
    e, count = np.zeros(1), 0
    for lv in levels:
        lv = lv[:np.searchsorted(lv, de * W.EV) + 1]
        s = e[:, None] + lv[None, :]
        count += int((s >= de * W.EV).any(axis=1).sum())
        e = s[s < de * W.EV]
    assert n == count + len(e)

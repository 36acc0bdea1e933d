"""Reaction counts summed on the host (up to 512 cells) and on the device:
against the cells' counters."""
import numpy as np
import pytest

from paper_2606_31548_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cells", [1, 511, 512, 513, 1000])
def test_reaction_counts(cells):
    from paper_2606_31548_amd import hcao
    wl = W.methane_chemistry(n_cells=cells, per_cell=64, t=20000.0, seed=cells)
    g = hcao.from_workload(wl)
    g.init_thermal(wl.counts, wl.t_trans, wl.t_vib)
    g.step(wl.dt, 20)
    want = g.cell_state()[2].sum(0)[hcao.CTR_REACTION0:hcao.CTR_REACTION0 + len(wl.reactions)]
    assert np.array_equal(g.reaction_counts(), want) and want.any()

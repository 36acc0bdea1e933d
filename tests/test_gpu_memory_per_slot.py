"""Device memory of a loaded context per particle slot: the state, and per work
entry (half as many) the staged product, the work list, the pair's velocities
and its records."""
import pytest

from paper_2606_31548_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("recombination", [False, True])
def test_bytes_per_slot(precision, recombination):
    import torch
    from paper_2606_31548_amd import hcao
    wl = W.methane_chemistry(n_cells=4000, per_cell=64, recombination=recombination)
    wl.capacity_per_cell = 2000
    warm = hcao.from_workload(wl, precision=precision)  # the library's module and tables
    warm.init_thermal(wl.counts, wl.t_trans, wl.t_vib)
    warm.close()
    g = hcao.from_workload(wl, precision=precision)
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    g.init_thermal(wl.counts, wl.t_trans, wl.t_vib)
    g.step(wl.dt, 1)
    g.sync()
    used = (free - torch.cuda.mem_get_info()[0]) / (4000 * 2000)
    row = 20  # nine modes
    body, pair, defect = (16, 24, 8) if precision else (32, 48, 0)
    want = (body + row) + ((body + row) + 32 + 1 + pair + defect + (40 if recombination else 0)) / 2
    assert abs(used - want) < 0.03 * want, (used, want)

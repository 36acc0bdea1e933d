"""Device scratch of the exact recombination sum: small ones stay with the
context, one of more than 512 MiB is given back."""
import numpy as np
import pytest

from paper_2606_31548_amd import workloads as W

pytestmark = pytest.mark.gpu


def test_large_scratch_is_given_back():
    import torch
    from paper_2606_31548_amd import hcao
    # five different soft bends: 60 M records of 12 bytes
    wl = W.methane_argon(n_cells=1, per_cell=16)
    wl.species = [W.Species("X", 44 * W.AMU, bend_theta_K=[37.0, 37.1, 37.2, 37.3, 37.4])]
    wl.reactions = []
    g = hcao.from_workload(wl)
    g.recombination_exact(0, 0.05 * W.EV, 0.74, np.array([3000.0]))
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    p, _, n = g.recombination_exact(0, 0.3 * W.EV, 0.74, np.array([3000.0]))
    assert 0.0 < p[0] < 1.0 and n * 12 > 512 << 20, n
    assert free - torch.cuda.mem_get_info()[0] < 64 << 20

"""Velocities and species of a checkpoint, converted on the device: the file's
arrays against the particles read back, and the restored state, below and above
the number of slots converted at a time (4,194,304)."""
import numpy as np
import pytest

from paper_2606_31548_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hc():
    from paper_2606_31548_amd import hcao
    hcao.load_library()
    return hcao


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("cells,per_cell,capacity", [(3, 41, 0), (20001, 30, 211)])
def test_checkpoint_bodies(hc, tmp_path, precision, cells, per_cell, capacity):
    wl = W.methane_argon(n_cells=cells, per_cell=per_cell, seed=6)
    wl.capacity_per_cell = capacity
    g = hc.from_workload(wl, precision=precision)
    g.init_thermal(wl.counts, wl.t_trans, wl.t_vib)
    g.step(wl.dt, 3)
    path = tmp_path / "state"
    g.save(path)
    counts, species, vel, levels = g.read_particles()
    # header of seven words; per cell: capacity, count, three numbers, counters; then the slots' arrays
    raw = path.read_bytes()
    tot = int(np.frombuffer(raw, np.uint64, 7)[3])
    cap = np.frombuffer(raw, np.uint32, cells, 56).astype(np.int64)
    assert tot == cap.sum() and (capacity == 0 or tot > 1 << 22)
    at = 56 + 8 * cells + 24 * cells + 8 * hc.N_CTR * cells
    used = np.arange(tot) - np.repeat(np.cumsum(cap) - cap, cap) < np.repeat(counts, cap)
    for k in range(3):
        v = np.frombuffer(raw, np.float64, tot, at + 8 * k * tot)
        assert np.array_equal(v[used].view(np.uint64), vel[:, k].copy().view(np.uint64))
    assert np.array_equal(np.frombuffer(raw, np.uint8, tot, at + 24 * tot)[used], species)
    b = hc.from_workload(wl, precision=precision)
    b.restore(path)
    for x, y in zip((counts, species, vel, levels), b.read_particles()):
        assert np.array_equal(x, y)
    c = cells // 2
    lo = int(counts[:c].sum())
    for n in (0, 1, int(counts[c]), 1 << 12):
        s, v, l = b.read_cell(c, max_n=n)
        k = min(n, int(counts[c]))
        assert np.array_equal(s, species[lo:lo + k]) and np.array_equal(v, vel[lo:lo + k])
        assert np.array_equal(l, levels[lo:lo + k])
    g.step(wl.dt, 2)
    b.step(wl.dt, 2)
    for x, y in zip(g.read_particles(), b.read_particles()):
        assert np.array_equal(x, y)

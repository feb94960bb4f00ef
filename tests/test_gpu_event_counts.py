"""The counts of reflections, kept on several lines of the device status: they add up
to the particles' event codes and survive everything that saves or restores them."""
import numpy as np
import pytest

import workloads
from gpu_helpers import require_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dpd():
    require_gpu()
    import paper_1807_09896_amd as dpd
    dpd.load_library()
    return dpd


def _counts(sim):
    c = sim.counters()
    return c["bounce"], c["fallback"]


# tiles of 256 particles: one, about eight, and more than the 64 lines
@pytest.mark.parametrize("L", [(4.0, 7.0, 4.0), (9.0, 8.0, 9.0), (24.0, 20.0, 24.0)])
def test_counts(dpd, L):
    s = workloads.slab_system(L=L, seed_fluid=21, seed_wall=22, grid_dtype=np.float32,
                              params=workloads.default_params(seed=23))
    print("event counts", s.n, flush=True)
    sim = dpd.Simulation(s)
    total = np.zeros(2, np.int64)
    for _ in range(12):
        sim.step(1)
        ev = sim.state()["events"]
        total += [int((ev == 1).sum()), int((ev == 2).sum())]
        assert _counts(sim) == tuple(total)
    assert total[0] > 0
    blob = sim.snapshot()
    sim.autotune(2)
    assert _counts(sim) == tuple(total)
    with pytest.raises(dpd.DPDError):
        sim.set_phi(-np.ones_like(np.asarray(s.phi)))
    assert _counts(sim) == tuple(total)
    sim.step(5)
    after = _counts(sim)
    sim.restore(blob)
    assert _counts(sim) == tuple(total)
    sim.step(5)
    assert _counts(sim) == after
    sim.close()

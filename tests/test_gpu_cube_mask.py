"""The mask of grid cubes next to the interface against numpy, on grids whose
cubes fill no whole word or wavefront (fewer than 32 cubes, and remainders of
each), at create and after the phase field is replaced."""
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


def _flagged(phi):
    neg = np.zeros(phi.shape, bool)
    for dz in (0, 1):
        for dy in (0, 1):
            for dx in (0, 1):
                neg |= np.roll(phi, (-dz, -dy, -dx), axis=(0, 1, 2)) < 0
    return int(neg.sum())


@pytest.mark.parametrize("dtype", [np.float32, np.float64], ids=["f32", "f64"])
@pytest.mark.parametrize("n", [(2, 3, 4), (4, 4, 4), (5, 7, 9), (33, 3, 21), (64, 16, 8)], ids=str)
def test_mask_matches_numpy(dpd, n, dtype):
    rng = np.random.default_rng(sum(n))
    L = np.array([4.0, 4.0, 4.0])
    s = workloads.bulk_system(L=tuple(L), seed=2)
    s.type = np.ones_like(s.type)          # walls only: any phase field is accepted
    s.vel = np.zeros_like(s.vel)
    s.h = L / np.array(n)
    fields = [np.where(rng.random(n[::-1]) < p, -0.5, 0.5).astype(dtype) for p in (0.02, 0.3, 0.0)]
    s.phi = fields[0]
    print("cube mask", n, dtype.__name__, flush=True)
    sim = dpd.Simulation(s)
    assert sim.counters()["mask_cells"] == _flagged(fields[0])
    for f in fields[1:]:
        sim.set_phi(f)
        assert sim.counters()["mask_cells"] == _flagged(f)
    sim.close()

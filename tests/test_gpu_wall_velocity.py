"""The search for a moving wall's velocity, shared by the lanes of a wavefront: one step
against the oracle with one, some and most of a wavefront's particles reflecting."""
import pytest

from gpu_helpers import require_gpu
from test_gpu_parity import _one_step_compare
from test_gpu_walls import _aimed_couette

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dpd():
    require_gpu()
    import paper_1807_09896_amd as dpd
    dpd.load_library()
    return dpd


@pytest.mark.parametrize("speed,band", [(1.5, 0.02), (12.0, 0.12), (45.0, 0.5)])
def test_reflections_per_wavefront(dpd, oracle_lib, speed, band):
    s = _aimed_couette(False, seed=71, speed=speed, band=band)
    sim = dpd.Simulation(s)
    sim.step(1)
    print("reflecting", speed, band, int((sim.state()["events"] > 0).sum()), "of", s.n, flush=True)
    sim.close()
    _one_step_compare(dpd, oracle_lib, s)

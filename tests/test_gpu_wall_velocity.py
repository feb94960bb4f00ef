"""Moving walls: the search for the wall nearest to a reflection, shared by the lanes of a
wavefront (one, some and most of a wavefront's particles reflecting), and the cell
list of fluid and walls together around the edges of its scan's chunks of 4,096 cells."""
import numpy as np
import pytest

import workloads
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


@pytest.mark.parametrize("L", [(16.0, 16.0, 16.0), (17.0, 16.0, 16.0), (16.0, 15.0, 17.0),
                               (24.0, 24.0, 15.0)])
def test_list_of_fluid_and_walls(dpd, oracle_lib, L):
    """One, one past, less than one and about two chunks; walls in every box's last cells
    too, and steps enough that walls change cells."""
    import torch
    s = workloads.couette_system(L=L, U=4.0, seed=73)
    print("list of fluid and walls", L, s.n, flush=True)
    _one_step_compare(dpd, oracle_lib, s, nsteps_before=2)
    small = _aimed_couette(True, seed=74)
    alone, batch = dpd.Simulation(s), dpd.Simulation([small, s], graph=True)
    for _ in range(3):
        alone.step(9)
        batch.step(9)
        a, b = alone.state(0), batch.state(1)
        for k in a:
            assert torch.equal(a[k], b[k]), k
        assert torch.equal(alone.forces(0), batch.forces(1))
    # the list built from the state (the walls listed apart) continues alike
    copy = dpd.Simulation(s)
    st = alone.state()
    copy.set_state(st["pos"], st["vel"], alone.forces(), alone.counters()["k"])
    pa, pb = alone.pairs(0), copy.pairs(0)
    order = lambda p: p[np.lexsort((p[:, 1], p[:, 0]))]
    assert np.array_equal(order(np.asarray(pa.cpu() if hasattr(pa, "cpu") else pa)),
                          order(np.asarray(pb.cpu() if hasattr(pb, "cpu") else pb)))
    for q in (alone, batch, copy):
        q.close()

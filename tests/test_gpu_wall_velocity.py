"""Moving walls: the search for the wall nearest to a reflection, shared by the lanes of a
wavefront (one, some and most of a wavefront's particles reflecting), and the cell
list of fluid and walls together around the edges of its scan's chunks of 1,024 cells,
and, from 2^20 cells on, of 4,096."""
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


@pytest.mark.parametrize("spec", [False, True])
def test_reflections_with_a_float64_grid(dpd, oracle_lib, spec):
    s = _aimed_couette(spec, seed=75, speed=20.0, band=0.25)
    s.phi = s.phi.astype(np.float64)
    _one_step_compare(dpd, oracle_lib, s)
    _one_step_compare(dpd, oracle_lib, s, nsteps_before=3)


@pytest.mark.parametrize("L", [(16.0, 8.0, 8.0), (31.0, 3.0, 11.0), (5.0, 5.0, 41.0),
                               (16.0, 16.0, 16.0), (17.0, 16.0, 16.0), (16.0, 15.0, 17.0),
                               (24.0, 24.0, 15.0)])
def test_list_of_fluid_and_walls(dpd, oracle_lib, L):
    """One chunk, one cell less and one past; four, and between them and eight; walls in every
    box's last cells too, and steps enough that walls change cells."""
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


@pytest.mark.parametrize("edge", [-1, 0, 1])
def test_list_of_fluid_and_walls_in_large_chunks(dpd, edge):
    """From 2^20 cells on the scan takes 4,096 cells a block: moving walls in such a context
    (256 such chunks, a cell less, which still takes chunks of 1,024, and some past) and alone,
    the same bits, with the box's cells across the edges of chunks."""
    from types import SimpleNamespace
    import torch
    s = workloads.couette_system(L=(21.0, 19.0, 12.0), U=4.0, seed=77)   # 4,788 cells
    rest = (1 << 20) - 2 * 4788
    # an almost empty box of the other cells: rest + edge = x y z
    x, y, z = {-1: (13, 3, rest // 39), 0: (5, 8, rest // 40), 1: (4, 4, rest // 16 + 1)}[edge]
    cells = x * y * z + 2 * 4788
    assert (cells < 1 << 20) == (edge < 0) and abs(cells - (1 << 20)) < 64
    n = 200
    rng = np.random.default_rng(78)
    L = np.array([x, y, z], dtype=np.float64)
    filler = SimpleNamespace(
        L=L, pos=(rng.random((n, 3)) * L * 0.999).astype(np.float32),
        vel=np.zeros((n, 3), np.float32), type=np.zeros(n, np.int32),
        gid=np.arange(n, dtype=np.uint32), phi=np.ones((2, 2, 2), np.float32), h=L / 2,
        params=dict(workloads.default_params(seed=79), replica=3))
    print("large chunks", edge, cells, s.n, flush=True)
    other = workloads.couette_system(L=(21.0, 19.0, 12.0), U=-3.0, seed=80)
    alone = [dpd.Simulation(s), dpd.Simulation(other)]
    batch = dpd.Simulation([s, filler, other])
    for n_ in (1, 1, 7):
        for sim in (*alone, batch):
            sim.step(n_)
        for r, sim in ((0, alone[0]), (2, alone[1])):
            a, b = sim.state(0), batch.state(r)
            for k in a:
                assert torch.equal(a[k], b[k]), (edge, n_, r, k)
            assert torch.equal(sim.forces(0), batch.forces(r)), (edge, n_, r)
    for sim in (*alone, batch):
        sim.close()

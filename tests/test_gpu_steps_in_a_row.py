"""Steps that follow one another in a call (the pair kernel goes on to the next drift)
against the same steps one call each, bit for bit, and captured steps replayed between
such calls, which exchange buffers that the captured steps hold."""
import numpy as np
import pytest

import workloads
from gpu_helpers import replay, require_gpu
from test_gpu_small_contexts import _edge_box, _sph
from test_gpu_walls import _aimed_couette

pytestmark = pytest.mark.gpu

P = workloads.default_params


@pytest.fixture(scope="module")
def dpd():
    require_gpu()
    import paper_1807_09896_amd as dpd
    dpd.load_library()
    return dpd


def _slab_of(L, dtype, seed):
    return workloads.slab_system(L=L, seed_fluid=seed, seed_wall=seed + 1, grid_dtype=dtype,
                                 params=P(seed=seed))


def _slab(dtype, seed):
    return _slab_of((9.0, 8.0, 9.0), dtype, seed)


CASES = {
    # 16 blocks per box, float32 and float64 grids
    "float32": lambda: [_slab(np.float32, 31)],
    "float64": lambda: [_slab(np.float64, 33)],
    "sph": lambda: [_sph(workloads.sinusoid_slit_system(L=(12.0, 8.0, 12.0), base=3.0, amp=1.0))],
    # one block per box, whose launch clears the counts itself
    "one_block": lambda: [_edge_box((7, 8, 6), 900 + 37 * r) for r in range(3)],
    "uneven": lambda: [_edge_box((4, 4, 4), 1), _slab(np.float32, 35), _edge_box((6, 5, 4), 1300)],
    # one lane per particle: the four launches of the cell list, its one launch (16 and 12
    # blocks a box), a box of part-filled wavefronts, float64
    "large": lambda: [_slab_of((36.0, 36.0, 24.0), np.float32, 41)],
    "large64": lambda: [_slab_of((36.0, 36.0, 24.0), np.float64, 43)],
    "large_sph": lambda: [_sph(workloads.sinusoid_slit_system(L=(36.0, 36.0, 24.0), base=3.0,
                                                              amp=1.0))],
    "batch16": lambda: [_slab_of((18.0, 26.0, 18.0 + 0.5 * r), np.float32, 45 + r)
                        for r in range(4)],
    "batch12": lambda: [_edge_box((12, 11, 10), 3400 + 13 * r) for r in range(20)],
    # moving walls (listed with the fluid on the way) alone and beside resting ones, and
    # specular reflection
    "large_moving": lambda: [workloads.couette_system(L=(41.0, 40.0, 17.5), U=4.0, seed=61)],
    "mixed_moving": lambda: [workloads.couette_system(L=(41.0, 40.0, 12.0), U=4.0, seed=62),
                             _slab_of((30.0, 29.0, 24.0), np.float32, 63)],
    "large_specular": lambda: [workloads.couette_system(L=(41.0, 40.0, 17.5), U=0.0, seed=64,
                                                        specular=True)],
    "moving_specular": lambda: [workloads.couette_system(L=(41.0, 40.0, 17.5), U=4.0, seed=65,
                                                         specular=True)],
    # the same in small contexts: a part-filled last wavefront, many reflections
    "moving": lambda: [workloads.couette_system(L=(8.0, 6.0, 7.0), U=4.0, seed=66)],
    "moving_aimed": lambda: [_aimed_couette(False, seed=67, speed=45.0, band=0.5)],
    "moving_batch": lambda: [workloads.couette_system(L=(8.0, 6.0, 7.0 + 0.5 * r), U=4.0,
                                                      seed=68 + r, specular=r == 1)
                             for r in range(3)] + [_slab(np.float32, 72)],
    "specular": lambda: [workloads.couette_system(L=(8.0, 6.0, 7.0), U=0.0, seed=36, specular=True)],
    # and with float64 grids
    "large_moving64": lambda: [workloads.couette_system(L=(41.0, 40.0, 17.5), U=4.0, seed=73,
                                                        specular=True, grid_dtype=np.float64)],
    "moving64": lambda: [workloads.couette_system(L=(8.0, 6.0, 7.0), U=4.0, seed=74,
                                                  grid_dtype=np.float64)],
    "specular64": lambda: [workloads.couette_system(L=(8.0, 6.0, 7.0), U=0.0, seed=75,
                                                    specular=True, grid_dtype=np.float64)],
}


@pytest.mark.parametrize("graph", [False, True])
@pytest.mark.parametrize("name", list(CASES))
def test_same_bits(dpd, name, graph):
    import torch
    boxes = CASES[name]()
    print("steps in a row", name, graph, [s.n for s in boxes], flush=True)
    one, row = dpd.Simulation(boxes), dpd.Simulation(boxes, graph=graph)

    def same(what):
        assert one.counters() == row.counters(), what
        for r in range(len(boxes)):
            a, b = one.state(r), row.state(r)
            for k in a:
                assert torch.equal(a[k], b[k]), (what, r, k)
            assert torch.equal(one.forces(r), row.forces(r)), (what, r)
            assert one.pairs(r).shape == row.pairs(r).shape, (what, r)

    for n in (2, 3, 1, 4, 7, 2):
        for _ in range(n):
            one.step(1)
        row.step(n)
        same(n)
    # a restored state goes on alike, and so does one after set_params
    blob = row.snapshot()
    row.step(5)
    row.restore(blob)
    one.step(1)
    one.step(1)
    row.step(2)
    same("restored")
    row.kernel_times(1)
    row.step(3)
    row.kernel_times(0)
    for _ in range(3):
        one.step(1)
    same("timed")
    one.close()
    row.close()


@pytest.mark.parametrize("name", ["one_block", "float32", "batch12", "large", "moving",
                                  "moving_batch", "large_moving"])
def test_replays_between_rows(dpd, name):
    """Steps captured from either buffer set and replayed before and after calls of several
    steps, which exchange the predictions and counts once or twice (and the buffer sets), and
    before and after the persistent step, against direct launches of single steps."""
    import torch
    boxes = CASES[name]()
    print("replays between rows", name, [s.n for s in boxes], flush=True)
    one, both = dpd.Simulation(boxes), dpd.Simulation(boxes, graph=True)
    moving = "moving" in name
    for turn, row in enumerate((0, 2, 3, 2, 2, 4, 3, 5, 0)):
        if row:
            both.step(row)
            replay(one, row)
        if turn == 5 and not moving:   # the persistent step's arguments hold one of each pair
            both.use_persistent(True)
            replay(both, 2)
            both.step(3)
            both.use_persistent(False)
            replay(one, 5)
        replay(both, 3)
        replay(one, 3)
        assert one.counters() == both.counters(), (turn, row)
        for r in range(len(boxes)):
            a, b = one.state(r), both.state(r)
            for k in a:
                assert torch.equal(a[k], b[k]), (turn, row, r, k)
            assert torch.equal(one.forces(r), both.forces(r)), (turn, row, r)
    one.close()
    both.close()

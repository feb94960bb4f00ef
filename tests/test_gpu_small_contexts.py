"""The kernels of small contexts against those of large ones, bit for bit.

A context of at most 65,536 fluid particles takes its pair forces with 16 lanes
per particle, and one whose boxes all fit in a block's LDS builds its cell lists
in one launch.  The same box beside a large one runs the kernels of large
contexts, and every result has to be the same: state, forces, events, pairs.
"""
import numpy as np
import pytest

import workloads
from gpu_helpers import replay as replay_steps
from gpu_helpers import require_gpu, sorted_pairs

pytestmark = pytest.mark.gpu

P = workloads.default_params


@pytest.fixture(scope="module")
def dpd():
    require_gpu()
    import paper_1807_09896_amd as dpd
    dpd.load_library()
    return dpd


@pytest.fixture(scope="module")
def filler():
    return workloads.bulk_system(L=(31.0, 30.0, 30.0), seed=91,
                                 params=P(seed=92, replica=7))


def _edge_box(cells, fluid):
    """A wall-free box of the given cell counts and fluid particles."""
    L = tuple(float(c) for c in cells)
    s = workloads.bulk_system(L=L, rho=1.02 * fluid / np.prod(L) + 0.01, seed=95,
                              params=P(seed=96))
    assert s.n >= fluid
    s.pos, s.vel, s.type = s.pos[:fluid], s.vel[:fluid], s.type[:fluid]
    s.gid = np.random.default_rng(97).permutation(fluid).astype(np.uint32)
    return s


def _squeezed():
    """1,400 particles in one corner of an otherwise empty box of 1,331 cells."""
    s = _edge_box((11, 11, 11), 1400)
    s.pos[:] = np.mod(s.pos * np.float32(0.27), np.float32(3.0))
    s.params = dict(s.params, a=[[0.5, 0.5], [0.5, 0.5]], dt=0.002)
    return s


def _sph(s):
    s.params = dict(s.params, sph=workloads.sph_force(), kBT=0.5, dt=0.005)
    return s


BOXES = {
    # three cells an axis: every cell is at both edges of its rows
    "three_cells": lambda: workloads.bulk_system(L=(3.0, 3.5, 3.5), seed=3, params=P(seed=4)),
    # one particle; 16 and 17 pairs lie around the size of one evaluation
    "single": lambda: _edge_box((4, 4, 4), 1),
    "sparse": lambda: _edge_box((6, 5, 4), 40),
    # 30 particles a cell: 650 candidates a particle, six rounds of 128
    "dense": lambda: workloads.bulk_system(L=(4.0, 5.0, 4.5), rho=24.0, seed=5,
                                           params=P(seed=6, a_ff=5.0, a_fs=5.0, dt=0.004)),
    "rc15": lambda: workloads.slab_system(L=(9.0, 8.0, 9.0), seed_fluid=11, seed_wall=12,
                                          grid_dtype=np.float32, params=dict(P(seed=13), rc=1.5)),
    "slab": lambda: workloads.tiny_slab_system(seed=14),
    "sph": lambda: _sph(workloads.sinusoid_slit_system(L=(12.0, 8.0, 12.0), base=3.0, amp=1.0)),
    "couette": lambda: workloads.couette_system(L=(8.0, 6.0, 7.0), seed=15, specular=True),
    # the largest box of the one-launch cell list, in particles and in cells,
    # and one past each
    "fluid_max": lambda: _edge_box((18, 18, 19), 24576),
    "fluid_over": lambda: _edge_box((18, 18, 19), 24577),
    "cells_max": lambda: _edge_box((32, 32, 16), 9000),
    "cells_over": lambda: _edge_box((33, 32, 16), 9000),
    # either side of one block per box
    "part_one": lambda: _edge_box((7, 8, 6), 1024),
    "part_many": lambda: _edge_box((7, 8, 6), 1025),
    # all particles in a few cells of one block's part of the box
    "corner": lambda: _squeezed(),
}


@pytest.mark.parametrize("name", list(BOXES))
def test_small_context_bits(dpd, filler, name):
    import torch
    s = BOXES[name]()
    print("small context", name, s.n, "particles, edges", s.L, flush=True)
    alone, beside = dpd.Simulation(s), dpd.Simulation([filler, s])
    for steps in (0, 1, 6):
        alone.step(steps)
        beside.step(steps)
        a, b = alone.state(0), beside.state(1)
        for k in a:
            assert torch.equal(a[k], b[k]), (name, steps, k)
        assert torch.equal(alone.forces(0), beside.forces(1)), (name, steps)
    pa, pb = alone.pairs(0), beside.pairs(1)
    assert np.array_equal(sorted_pairs(pa), sorted_pairs(pb))
    alone.close()
    beside.close()


@pytest.mark.parametrize("count,fluid", [(3, 1100), (70, 1100), (130, 1100), (512, 200),
                                         (513, 200), (513, 1536)])
def test_blocks_per_box(dpd, count, fluid):
    """Batches whose boxes are shared by 16, 3 and one block each; above 512 boxes only
    large ones take the one launch."""
    import torch
    cells = (7, 8, 6) if fluid < 1500 else (8, 8, 8)
    boxes = [_edge_box(cells, fluid + 3 * (r % 140)) for r in range(count)]
    print("blocks per box", count, fluid, flush=True)
    batch = dpd.Simulation(boxes)
    batch.kernel_times(1)
    batch.step(1)
    scans = batch.kernel_times(0)["scan_down"][1]
    assert scans == (1 if count > 512 and fluid < 1500 else 0)
    batch.step(3)
    for r in (0, count // 2, count - 1):
        alone = dpd.Simulation(boxes[r])
        alone.step(4)
        a, b = alone.state(0), batch.state(r)
        for k in a:
            assert torch.equal(a[k], b[k]), (count, r, k)
        alone.close()
    # counts are clear again after calls that build a list without a force
    assert batch.pairs(0).shape == batch.pairs(0).shape
    batch.step(2)
    batch.sync()
    batch.close()


@pytest.mark.parametrize("count,walls", [(3, False), (4, True), (20, False)])
def test_codes_of_the_box_list(dpd, count, walls):
    """Contexts above the 16-lane pair kernel's size whose coarse codes the cell
    list's own 16 blocks per box write, and (20 boxes, 12 blocks) a launch after it."""
    import torch
    boxes = []
    for r in range(count):
        if walls:
            boxes.append(workloads.slab_system(L=(18.0, 26.0, 18.0 + 0.5 * r), seed_fluid=30 + r,
                                               seed_wall=50 + r, grid_dtype=np.float32,
                                               params=P(seed=r)))
        else:
            boxes.append(_edge_box((18, 18, 19), 24576 - r) if count < 16 else
                         _edge_box((12, 11, 10), 3500 + r))
    fluid = sum(int((s.type == 0).sum()) for s in boxes)
    print("codes", count, walls, fluid, flush=True)
    assert fluid > 65536
    batch = dpd.Simulation(boxes)
    batch.step(5)
    for r in (0, count - 1):
        alone = dpd.Simulation(boxes[r])
        alone.step(5)
        a, b = alone.state(0), batch.state(r)
        for k in a:
            assert torch.equal(a[k], b[k]), (count, r, k)
        assert torch.equal(alone.forces(0), batch.forces(r)), (count, r)
        alone.close()
    batch.close()


def test_small_context_graph_replays(dpd):
    """The small context's step captured and replayed, eager work between."""
    import torch
    s = BOXES["slab"]()
    direct, replay = dpd.Simulation(s), dpd.Simulation(s, graph=True)
    for k in range(6):
        direct.step(3)
        replay_steps(replay, 3)
        a, b = direct.state(), replay.state()
        for q in a:
            assert torch.equal(a[q], b[q]), (k, q)
        assert torch.equal(direct.forces(), replay.forces()), k
    direct.close()
    replay.close()

"""Rows of the per-box getters: every gid written once, fluid and walls, whatever
the buffers held, for box sizes around the edges of a block."""
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


def _box(nf, nw, seed):
    """nf fluid particles and nw walls on a lattice, gids shuffled."""
    L = (12.0, 12.0, 12.0)
    side = np.arange(12, dtype=np.float32) + np.float32(0.5)
    pos = np.stack(np.meshgrid(side, side, side, indexing="ij"), -1).reshape(-1, 3)
    rng = np.random.default_rng(seed)
    s = workloads.bulk_system(L=L, rho=3.0, seed=seed, params=workloads.default_params(seed=seed))
    n = nf + nw
    assert n <= len(pos) and n <= s.n
    s.pos = np.ascontiguousarray(pos[rng.permutation(len(pos))[:n]])
    s.vel = rng.uniform(-1, 1, (n, 3)).astype(np.float32)
    s.type = np.zeros(n, np.int32)
    s.type[rng.permutation(n)[:nw]] = 1
    s.vel[s.type == 1] = 0
    s.gid = rng.permutation(n).astype(np.uint32)
    return s


@pytest.mark.parametrize("nf,nw", [(1, 0), (1, 1), (255, 1), (256, 0), (256, 256), (257, 254),
                                   (640, 1)])
def test_rows(dpd, nf, nw):
    import torch
    from paper_1807_09896_amd import binding
    print("getter rows", nf, nw, flush=True)
    boxes = [_box(nf, nw, 5), _box(300, 7, 6)]
    sim = dpd.Simulation(boxes)
    for r, s in enumerate(boxes):
        n = len(s.pos)
        pos = torch.full((n, 3), np.nan, device="cuda")
        vel, frc = pos.clone(), pos.clone()
        ev = torch.full((n,), -7, dtype=torch.int32, device="cuda")
        cell = ev.clone()
        binding.dpd_replica_state(sim.ctx, r, pos, vel, ev, cell)
        binding.dpd_replica_forces(sim.ctx, r, frc)
        order = np.argsort(s.gid)
        assert np.array_equal(pos.cpu().numpy(), s.pos[order])
        assert np.array_equal(vel.cpu().numpy(), s.vel[order])
        assert not ev.any()
        c = np.floor(s.pos[order]).astype(int)
        assert np.array_equal(cell.cpu().numpy(), (c[:, 2] * 12 + c[:, 1]) * 12 + c[:, 0])
        walls = torch.from_numpy(s.type[order] == 1).cuda()
        assert torch.isfinite(frc).all() and not frc[walls].any()
        # each output alone, the others not asked for
        for k, ref in enumerate((pos, vel, ev, cell)):
            one = torch.full_like(ref, -3)
            binding.dpd_replica_state(sim.ctx, r, *[one if q == k else None for q in range(4)])
            assert torch.equal(one, ref), k
    sim.close()

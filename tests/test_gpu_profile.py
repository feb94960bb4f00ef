"""dpd_profile against direct numpy binning of the state it is read from.

The bin of a particle is floor(fl(fl(x / L) nbins)) in FP32, so counts are
exact.  The sums are FP64 sums in an order of their own: n terms differ by at
most n 2^-53 of the sum of their magnitudes.
"""
import sys

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


def _bulk(edge, n_extra):
    """A wall-free box of edge^3 at density 3, with n_extra particles dropped
    so that the count is no multiple of a block."""
    s = workloads.bulk_system(L=(edge, edge + 1.0, edge + 2.0), seed=5)
    n = s.n - n_extra
    s.pos, s.vel, s.type = s.pos[:n], s.vel[:n], s.type[:n]
    s.gid = np.random.default_rng(6).permutation(n).astype(np.uint32)
    return s


# 1,019 particles (one block), 300 blocks' worth of 1,024 (more than the 256
# launched) and a slab whose bins at the walls stay empty
@pytest.mark.parametrize("which", ["small", "large", "slab"])
def test_profile_matches_numpy(dpd, which):
    s = {"small": lambda: _bulk(6.0, 3), "large": lambda: _bulk(46.0, 1),
         "slab": lambda: workloads.slab_system()}[which]()
    sim = dpd.Simulation(s)
    sim.step(2)
    st = sim.state()
    pos, vel = st["pos"].cpu().numpy(), st["vel"].cpu().numpy().astype(np.float64)
    typ = np.empty_like(s.type)
    typ[s.gid] = s.type
    pos, vel = pos[typ == 0], vel[typ == 0]
    for axis in (0, 1, 2):
        for nbins in (1, 2, 7, 64, 1024, 1025, 3000):
            print("profile", which, pos.shape[0], "axis", axis, "bins", nbins, flush=True)
            sys.stdout.flush()
            got = sim.profile(axis, nbins).cpu().numpy()
            f = np.floor(pos[:, axis] / np.float32(s.L[axis]) * np.float32(nbins))
            b = np.clip(f.astype(np.int64), 0, nbins - 1)
            cnt = np.bincount(b, minlength=nbins)
            assert np.array_equal(got[:, 0], cnt)
            cols = [vel[:, 0], vel[:, 1], vel[:, 2], (vel ** 2).sum(1)]
            for q, c in enumerate(cols):
                want = np.bincount(b, weights=c, minlength=nbins)
                size = np.bincount(b, weights=np.abs(c), minlength=nbins)
                assert np.all(np.abs(got[:, q + 1] - want) <= 2 * (cnt + 2) * 2.0 ** -53 * size), q
    sim.close()

"""The cell list's scan around the edges of its blocks (1,024 cells each, 4,096 from 2^20
cells on): pairs of sparse wall-free boxes against a k-d tree."""
import numpy as np
import pytest
from scipy.spatial import cKDTree

import workloads
from gpu_helpers import require_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dpd():
    require_gpu()
    import paper_1807_09896_amd as dpd
    dpd.load_library()
    return dpd


# cells: 17 blocks, one less, one more than 17 blocks, 2^20, 2^20 less a row, and above
@pytest.mark.parametrize("cells", [(32, 32, 17), (33, 31, 17), (43, 27, 15), (128, 128, 64),
                                   (127, 128, 64), (131, 128, 64)])
def test_pairs(dpd, cells):
    L = np.array(cells, float)
    count = int(np.prod(cells))
    print("cells", cells, count, flush=True)
    s = workloads.bulk_system(L=tuple(L), rho=0.1, seed=11,
                              params=workloads.default_params(seed=12))
    sim = dpd.Simulation(s)
    sim.step(2)
    st = sim.state()
    pos = st["pos"].cpu().numpy()
    cell = np.minimum(np.floor(pos).astype(int), np.array(cells) - 1)
    index = (cell[:, 2] * cells[1] + cell[:, 1]) * cells[0] + cell[:, 0]
    assert np.array_equal(st["cell_of"].cpu().numpy(), index)
    p = sim.pairs()
    p = np.asarray(p.cpu() if hasattr(p, "cpu") else p).astype(np.int64)
    got = np.unique(p[:, 0] * s.n + p[:, 1])
    assert len(got) == len(p)
    # positions just below an edge may round to it in the tree's wrap
    tree = cKDTree(np.mod(pos.astype(float), L), boxsize=L)

    def keys(r):
        q = tree.query_pairs(r, output_type="ndarray").astype(np.int64)
        return np.unique(np.concatenate([q[:, 0] * s.n + q[:, 1], q[:, 1] * s.n + q[:, 0]]))

    # FP32 decides distances within 1e-6 of the cutoff
    assert np.isin(keys(1.0 - 1e-6), got).all()
    assert np.isin(got, keys(1.0 + 1e-6)).all()
    assert len(got) > 0
    sim.close()

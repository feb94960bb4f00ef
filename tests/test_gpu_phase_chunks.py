"""Phase-field relaxation over the z-chunk sizes that a grid can get, against
the oracle: grids that take 4, 8, 12, 16 and 24 planes per block in one type or the
other, with chunks that end ragged (one plane left over), and fields without a
gradient, where the reciprocal of its length comes from its floor.

Tolerances as in the other relaxation tests: the unit roundoff times the 100-fold
amplification that these inputs are bounded by, with margin.
"""
import numpy as np
import pytest

import workloads
from gpu_helpers import require_gpu
from oracle import phase_field as pf

pytestmark = pytest.mark.gpu

EPS = 0.5 / np.sqrt(2.0)
TOL = {4: 1e-5, 8: 1e-12}


@pytest.fixture(scope="module")
def dpd():
    require_gpu()
    import paper_1807_09896_amd as dpd
    dpd.load_library()
    return dpd


def _relax(dpd, phi0, h, dtau, iters, dtype):
    import torch
    td = torch.float32 if dtype == 4 else torch.float64
    phi = torch.tensor(phi0, dtype=td, device="cuda")
    work = torch.empty(phi.numel() + 1, dtype=td, device="cuda")
    res = dpd.dpd_phi_relax(phi, work, h, EPS, dtau, iters)
    return phi.cpu().numpy().astype(np.float64), res


@pytest.mark.parametrize("dtype", [4, 8], ids=["f32", "f64"])
@pytest.mark.parametrize("n", [(65, 17, 9), (96, 128, 105), (187, 130, 97), (250, 200, 121),
                               (300, 250, 145)], ids=str)
def test_chunks_match_oracle(dpd, n, dtype):
    h = (0.25, 0.25, 0.25)
    phi0 = workloads.step_phase_field(n, h, seed=sum(n))
    dtau = 0.5 * pf.max_stable_dtau(h, EPS)
    print("relax chunks", n, "dtype", dtype, flush=True)
    ref, rres = pf.relax(phi0, h, EPS, dtau, 3)
    out, res = _relax(dpd, phi0, h, dtau, 3, dtype)
    assert np.abs(out - ref).max() <= TOL[dtype]
    assert abs(res - rres) <= TOL[dtype] * max(rres, 1.0)


@pytest.mark.parametrize("dtype", [4, 8], ids=["f32", "f64"])
def test_fields_without_gradient(dpd, dtype):
    h = (0.25, 0.25, 0.25)
    for value in (0.0, 1.0, -1.0, 0.5):
        phi0 = np.full((9, 20, 70), value)
        ref, rres = pf.relax(phi0, h, EPS, 0.01, 2)
        out, res = _relax(dpd, phi0, h, 0.01, 2, dtype)
        assert np.abs(out - ref).max() <= TOL[dtype], value
        assert abs(res - rres) <= TOL[dtype], value


@pytest.mark.parametrize("value,dtype", [(np.inf, 4), (np.inf, 8), (-np.inf, 8), (1e200, 8),
                                         (-1e158, 8), (np.nan, 4), (np.nan, 8)], ids=str)
def test_overflow_stays_where_it_is(dpd, monkeypatch, value, dtype):
    """One node of a smooth field infinite, NaN, or so large that a squared length overflows:
    after one step the same nodes are infinite and NaN as in the oracle, where a finite part
    over an infinite length is zero, and the others have its values.  (The floor of a length
    that is NaN is the floor in the kernel, as fmax has it.)"""
    nx, ny, nz = 70, 20, 9
    z, y, x = np.meshgrid(np.arange(nz), np.arange(ny), np.arange(nx), indexing="ij")
    phi0 = 0.6 * np.sin(0.3 * x + 0.2) * np.cos(0.45 * y + 0.7 * z) + 0.1 * np.sin(0.9 * z + 0.4 * y)
    phi0[4, 15, 63] = value   # beside a tile's edge in x and in y
    phi0 = phi0.astype(np.float32).astype(np.float64) if dtype == 4 else phi0
    h = (0.25, 0.25, 0.25)
    with np.errstate(all="ignore"), monkeypatch.context() as m:
        m.setattr(np, "maximum", np.fmax)
        ref, _ = pf.relax(phi0, h, EPS, 0.01, 1)
    print("relax overflow", value, dtype, int((~np.isfinite(ref)).sum()), flush=True)
    out, _ = _relax(dpd, phi0, h, 0.01, 1, dtype)
    assert np.array_equal(np.isnan(out), np.isnan(ref))
    assert np.array_equal(np.isposinf(out), np.isposinf(ref))
    assert np.array_equal(np.isneginf(out), np.isneginf(ref))
    near = np.abs(ref) < 1e6
    assert near.sum() > ref.size - 100
    assert np.abs(out[near] - ref[near]).max() <= TOL[dtype]

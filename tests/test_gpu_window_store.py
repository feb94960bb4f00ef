"""A window kept whole against one recomputed from its checkpoints.

A window whose steps fit 2 GiB is kept whole; one whose store cannot be
allocated keeps a state every ckpt steps and recomputes.  Both run the same
kernels on the same values, so profile, counts, scalar gradients and the final
state agree bit for bit; the phase-field gradient is summed by FP64 atomics, whose
order is free (1e-12 of its size).  Sizes on both sides of the 65,536 particles
up to which 16 lanes share a particle.
"""
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


def _window(dpd, s, steps, ckpt, monkeypatch, refuse):
    """refuse: allocations of at least so many bytes fail once the simulation exists, as
    torch's fail: with an exception."""
    import types
    import torch
    from paper_1807_09896_amd import binding
    from paper_1807_09896_amd.adjoint import Window
    made = []

    class Allocator(binding.TorchAllocator):
        limit, refused = None, 0

        def __init__(self, device):
            super().__init__(device)
            self._torch = types.SimpleNamespace(empty=self._empty, uint8=torch.uint8)
            made.append(self)

        def _empty(self, nbytes, **kw):
            if self.limit is not None and nbytes >= self.limit:
                self.refused += 1
                raise torch.cuda.OutOfMemoryError("refused")
            return torch.empty(nbytes, **kw)

    monkeypatch.setattr(binding, "TorchAllocator", Allocator)
    sim = dpd.Simulation(s, graph=True)
    monkeypatch.undo()
    win = Window(sim, steps=steps, ckpt=ckpt, axis=2, nbins=24)
    made[0].limit = refuse
    phi = torch.from_numpy(s.phi).to("cuda")
    p = dict(s.params, gamma=4.2, g=[0.03, 0.0, 0.0])
    weights = torch.linspace(-1.0, 1.0, 24, dtype=torch.float64, device="cuda")
    got = []
    for _ in range(2):   # a second window reuses the buffers
        prof = win.run(p, phi)
        grads, dphi = win.backward(weights)
        st = sim.state()
        got.append((prof.clone(), win.counts.clone(), grads, dphi.clone(), st["pos"], st["vel"],
                    sim.forces(), sim.counters()))
    refused = made[0].refused
    sim.step(3)   # the context goes on as it would
    last = sim.state()
    sim.close()
    return got, last, refused


@pytest.mark.parametrize("which,steps,ckpt", [("small", 1, 1), ("small", 7, 3), ("small", 12, 12),
                                              ("large", 5, 2)])
def test_kept_window_matches_recomputed(dpd, monkeypatch, which, steps, ckpt):
    import torch
    L = (12.0, 8.0, 12.0) if which == "small" else (36.0, 36.0, 24.0)
    s = workloads.sinusoid_slit_system(L=L, base=2.5, amp=1.0)
    assert (s.n_fluid > 65536) == (which == "large")
    print("window store", which, s.n, "steps", steps, "ckpt", ckpt, flush=True)
    kept, kept_last, none = _window(dpd, s, steps, ckpt, monkeypatch, None)
    # the store of `steps` steps is the largest buffer: about 100 bytes a particle and step,
    # beside at most 48 per checkpoint or segment state and 176 of adjoints
    limit = 80 * s.n_fluid * steps
    again, again_last, refused = _window(dpd, s, steps, ckpt, monkeypatch, limit) \
        if steps > 2 else (kept, kept_last, 1)
    assert none == 0 and refused > 0
    for k, a in zip(kept, again):
        for q in (0, 1, 4, 5, 6):
            assert torch.equal(k[q], a[q]), q
        assert k[2] == a[2]
        size = float(k[3].abs().max())
        assert float((k[3] - a[3]).abs().max()) <= 1e-12 * max(size, 1e-300)
        assert k[7] == a[7]
    for q in kept_last:
        assert torch.equal(kept_last[q], again_last[q]), q


def test_trace_of_a_kept_window(dpd):
    """dpd_window_trace of a kept window ends where the window ended."""
    import torch
    from paper_1807_09896_amd import binding
    s = workloads.sinusoid_slit_system(L=(12.0, 8.0, 12.0), base=2.5, amp=1.0)
    sim = dpd.Simulation(s)
    sim.step(2)
    binding.dpd_window_forward(sim.ctx, 7, 3, 2, 10)
    end = sim.state()
    pos = torch.empty((8, s.n, 3), device="cuda")
    ev = torch.empty((7, s.n), dtype=torch.int32, device="cuda")
    binding.dpd_window_trace(sim.ctx, pos_log=pos, ev_log=ev)
    after = sim.state()
    for q in end:
        assert torch.equal(end[q], after[q]), q
    assert torch.equal(pos[7], end["pos"]) and torch.equal(ev[6], end["events"])
    assert np.isfinite(binding.dpd_backward(
        sim.ctx, torch.ones(10, dtype=torch.float64, device="cuda"))).all()
    sim.close()

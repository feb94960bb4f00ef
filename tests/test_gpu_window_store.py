"""A window kept whole against one recomputed from its checkpoints.

A window whose steps fit 2 GiB is kept whole; one whose store cannot be
allocated keeps a state every ckpt steps and recomputes.  (Below: memory that only saves
time is done without, and given back, where an allocation fails.)  Both run the same
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


def _simulation(dpd, s, monkeypatch, refuse=None, **kw):
    """A simulation and its allocator, whose memory fails where refuse(bytes) holds, as
    torch's fails: with an exception."""
    import types
    import torch
    from paper_1807_09896_amd import binding
    made = []

    class Allocator(binding.TorchAllocator):
        def __init__(self, device):
            super().__init__(device)
            self._torch = types.SimpleNamespace(empty=self._empty, uint8=torch.uint8)
            self.refuse, self.refused, self.sizes = refuse, 0, []
            made.append(self)

        def _empty(self, nbytes, **kw):
            self.sizes.append(nbytes)
            if self.refuse and self.refuse(nbytes):
                self.refused += 1
                raise torch.cuda.OutOfMemoryError("refused")
            return torch.empty(nbytes, **kw)

        def held(self):
            return sum(t.numel() for t in self.live.values())

        def limit(self, total):
            self.refuse = lambda nbytes: self.held() + nbytes > total

    with monkeypatch.context() as m:
        m.setattr(binding, "TorchAllocator", Allocator)
        sim = dpd.Simulation(s, **kw)
    return sim, made[0]


def _step_bytes(s):
    """One step of a kept window: its state, drifted positions and predictions with walls and
    pad, the order and the merged runs, the run starts; each part in units of 256."""
    nf, rec = s.n_fluid, s.n + 1
    cells = int(np.prod(np.floor(np.asarray(s.L) / s.params["rc"])))
    parts = (48 * nf, 16 * rec, 16 * rec, 4 * nf, 4 * (rec - 1 + 8), 4 * (cells + 1 + 4))
    return sum((b + 255) // 256 * 256 for b in parts)


def _window(dpd, s, steps, ckpt, monkeypatch, refuse):
    """refuse: an allocation of so many bytes fails once the simulation exists."""
    import torch
    from paper_1807_09896_amd.adjoint import Window
    sim, alloc = _simulation(dpd, s, monkeypatch, graph=True)
    win = Window(sim, steps=steps, ckpt=ckpt, axis=2, nbins=24)
    if refuse:
        alloc.refuse = lambda nbytes: nbytes == refuse
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
    refused = alloc.refused
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
    again, again_last, refused = _window(dpd, s, steps, ckpt, monkeypatch, _step_bytes(s) * steps)
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


def test_store_goes_back(dpd, monkeypatch):
    """The store leaves with the first window that does not use it."""
    import torch
    from paper_1807_09896_amd import binding
    s = workloads.bulk_system(L=(9.0, 9.0, 9.0), seed=21, params=workloads.default_params(seed=21))
    sim, alloc = _simulation(dpd, s, monkeypatch)
    step = _step_bytes(s)
    binding.dpd_window_forward(sim.ctx, 40, 5, 2, 10)
    small = alloc.held()
    assert 40 * step in alloc.sizes
    steps = (1 << 31) // step + 1   # past 2 GiB by less than a step
    print("store goes back", s.n, steps, flush=True)
    binding.dpd_window_forward(sim.ctx, steps, 64, 2, 10)
    states = 48 * s.n_fluid * ((steps + 63) // 64 + 64)
    assert max(alloc.sizes) < 1 << 30
    assert alloc.held() <= small - 40 * step + states + 512
    # a small window is kept again, and swept (gradients over the large one's thousands of
    # chaotic steps exceed float32)
    binding.dpd_window_forward(sim.ctx, 40, 5, 2, 10)
    assert alloc.sizes.count(40 * step) == 2
    grads = binding.dpd_backward(sim.ctx, torch.ones(10, dtype=torch.float64, device="cuda"))
    assert np.isfinite(grads).all()
    sim.close()


MEMORY = {"one_block": lambda: workloads.bulk_system(L=(7.0, 7.0, 6.0), seed=22),
          "blocks": lambda: workloads.bulk_system(L=(10.0, 10.0, 10.0), seed=23),
          "large": lambda: workloads.bulk_system(L=(29.0, 29.0, 29.0), seed=24)}


@pytest.mark.parametrize("name", list(MEMORY))
def test_steps_without_second_buffers(dpd, monkeypatch, name):
    """A context is created, and steps alike, where the buffers that only save time (its last
    allocations) are refused."""
    import torch
    s = MEMORY[name]()
    want, alloc = _simulation(dpd, s, monkeypatch)
    want.step(7)
    a = want.state()
    count = len(alloc.sizes)
    spare = 2 if name != "large" else 1   # the prediction and, with the box list, the counts
    assert alloc.sizes[count - spare] == (16 * (s.n + 1) + 255) // 256 * 256
    for first in range(count - spare, count):
        seen = [0]

        def refuse(nbytes):
            seen[0] += 1
            return seen[0] > first
        sim, tried = _simulation(dpd, s, monkeypatch, refuse=refuse)
        assert tried.refused > 0
        sim.step(7)
        b = sim.state()
        for q in a:
            assert torch.equal(a[q], b[q]), (first, q)
        assert torch.equal(want.forces(), sim.forces()), first
        sim.close()
    want.close()


@pytest.mark.parametrize("how", ["direct", "graph", "persistent"])
@pytest.mark.parametrize("name", list(MEMORY))
def test_second_buffers_go_back(dpd, monkeypatch, name, how):
    """Where set_phi's memory is there only without the buffers that only save time, they
    go, and the context steps on alike: after an odd number of exchanges, with captured
    steps that held either, with the persistent step's arguments."""
    import torch
    s = MEMORY[name]()
    want, (sim, alloc) = dpd.Simulation(s), _simulation(dpd, s, monkeypatch, graph=how == "graph")
    assert s.phi.nbytes <= 16 * s.n
    for n in (1, 1, 2, 1, 2, 4):
        sim.step(n)
        want.step(n)
    if how == "persistent":
        sim.use_persistent(True)
        sim.step(1)
        want.step(1)
    held = alloc.held()
    alloc.limit(held)
    print("second buffers go back", name, how, s.n, held, flush=True)
    sim.set_phi(torch.from_numpy(s.phi).to("cuda"))
    assert alloc.refused == 1 and alloc.held() <= held - 16 * s.n
    for n in (1, 1, 3, 1, 2):
        sim.step(n)
        want.step(n)
        if how == "persistent" and n == 3:
            sim.use_persistent(False)
    a, b = want.state(), sim.state()
    for q in a:
        assert torch.equal(a[q], b[q]), q
    assert torch.equal(want.forces(), sim.forces())
    assert want.counters() == sim.counters()
    want.close()
    sim.close()


def test_second_buffers_stay_with_a_callers_graph(dpd, monkeypatch):
    """A graph that the caller captured holds the second buffers, so they stay: the call that
    would need their memory reports none, and the graph replays as before."""
    import torch
    s = MEMORY["blocks"]()
    side = torch.cuda.Stream()
    want = dpd.Simulation(s)
    sim, alloc = _simulation(dpd, s, monkeypatch, stream=side)
    side.synchronize()
    print("second buffers and a caller's graph", s.n, flush=True)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=side):
        sim.step(2)
    phi = torch.from_numpy(s.phi).to("cuda")
    torch.cuda.synchronize()
    alloc.limit(alloc.held())
    for _ in range(3):
        with pytest.raises(dpd.DPDError):
            sim.set_phi(phi)
        with torch.cuda.stream(side):
            g.replay()
        side.synchronize()
        want.step(2)
        a, b = want.state(), sim.state()
        for q in a:
            assert torch.equal(a[q], b[q]), q
    del g
    want.close()
    sim.close()

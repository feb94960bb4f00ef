"""The attractive-repulsive conservative force of Eq. 22-24 on the GPU,
through the C ABI.

Bars: forces at the initial state against the oracle within 2e-5 F_scale,
and one step from a common FP32 snapshot with the one-step bar of the
standard-force parity tests (events bit-exact, cells, positions,
velocities, forces), on a resting slab, a curved channel and a Couette slab
with a sliding plate; a batch that mixes boxes with and without the force
gives each box the bits it has alone, under graph replay too; switching the
force on with set_params during a graph-replayed run gives the bits of a
run with direct launches; a long run keeps the oracle's kinetic
temperature; the adjoint form refuses the force.
"""
import sys

import numpy as np
import pytest

import workloads
from gpu_helpers import by_gid, force_scale, replay, require_gpu
from test_gpu_parity import FORCE_TOL, _one_step_compare, _small_curved

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def dpd():
    require_gpu()
    import paper_1807_09896_amd as dpd
    dpd.load_library()
    return dpd


def _with_sph(s, kBT=0.5, dt=0.005, fs_factor=2.0):
    """Sec. IV's fluid: kBT = 0.5, gamma = 4.5, the Eq. 22-24 strengths and
    ranges, fluid-solid strengths twice the fluid-fluid ones."""
    p = dict(s.params)
    p["sph"] = workloads.sph_force(fs_factor=fs_factor)
    p["kBT"] = kBT
    p["dt"] = dt
    s.params = p
    return s


SYSTEMS = {
    "slab": lambda: _with_sph(workloads.tiny_slab_system()),
    "curved": lambda: _with_sph(_small_curved(seed=14)),
    "couette": lambda: _with_sph(workloads.couette_system(U=1.0, seed=90)),
}


@pytest.mark.parametrize("name", list(SYSTEMS))
def test_initial_forces(dpd, oracle_lib, name):
    s = SYSTEMS[name]()
    say("sph system", name, "n", s.n)
    o = oracle_lib.Oracle(s)
    sim = dpd.Simulation(s)
    f_gpu = sim.forces().cpu().numpy().astype(np.float64)
    f_or = by_gid(o, o.f)
    fluid = by_gid(o, s.type) == 0
    scale = force_scale(f_or[fluid])
    err = np.abs(f_gpu - f_or).max(axis=1)
    say("max err / F_scale", err[fluid].max() / scale)
    assert err[fluid].max() <= FORCE_TOL * scale
    assert np.all(f_gpu[~fluid] == 0)
    sim.close()


@pytest.mark.parametrize("name", list(SYSTEMS))
def test_one_step(dpd, oracle_lib, name):
    s = SYSTEMS[name]()
    say("sph one-step", name, s.n)
    _one_step_compare(dpd, oracle_lib, s)


def test_one_step_mid_run(dpd, oracle_lib):
    """Snapshot after 40 oracle steps: the state the force itself produced."""
    s = _with_sph(workloads.tiny_slab_system(seed=9))
    _one_step_compare(dpd, oracle_lib, s, nsteps_before=40)


def _snap(sim, r):
    st = {k: v.cpu().numpy() for k, v in sim.state(r).items()}
    st["force"] = sim.forces(r).cpu().numpy()
    return st


def _same(a, b, what):
    for k in ("pos", "vel", "events", "cell_of", "force"):
        assert np.array_equal(a[k], b[k]), (what, k)


def test_batch_mixing_forces_and_graph(dpd):
    boxes = [workloads.tiny_slab_system(seed=11),
             _with_sph(workloads.tiny_slab_system(seed=12)),
             _with_sph(workloads.couette_system(U=0.5, seed=91))]
    batch = dpd.Simulation(boxes)
    batch.step(15)
    for r in range(3):
        alone = dpd.Simulation(boxes[r])
        alone.step(15)
        _same(_snap(batch, r), _snap(alone, 0), ("batch vs alone", r))
        alone.close()
    graph = dpd.Simulation(boxes, graph=True)
    replay(graph, 15)
    for r in range(3):
        _same(_snap(graph, r), _snap(batch, r), ("graph", r))
    graph.close()
    batch.close()


def test_set_params_switches_the_force(dpd):
    """A graph captured without the force is dropped when set_params turns
    it on: the run matches one with direct launches."""
    s = workloads.tiny_slab_system(seed=13)
    on = _with_sph(workloads.tiny_slab_system(seed=13)).params
    runs = []
    for graph in (True, False):
        sim = dpd.Simulation(s, graph=graph)
        replay(sim, 6)
        sim.set_params(on)
        replay(sim, 6)
        runs.append(_snap(sim, 0))
        sim.close()
    _same(runs[0], runs[1], "graph vs direct")
    # and differs from the run that kept the linear force
    sim = dpd.Simulation(s)
    sim.step(12)
    assert not np.array_equal(_snap(sim, 0)["vel"], runs[1]["vel"])
    sim.close()


def test_kinetic_temperature_matches_oracle(dpd, oracle_lib):
    """A wetting film between resting plates (fluid-solid strengths twice
    the fluid-fluid ones): the kinetic temperature of a long run on the GPU
    agrees with the oracle's run of the same system (block means, 3 standard
    errors plus 0.01 for the state-dependent part that block means of one
    run do not sample)."""
    s = _with_sph(workloads.couette_system(L=(6.0, 6.0, 7.0), U=0.0, rho=3.0, seed=83))
    warm, blocks, per = 1500, 8, 50

    o = oracle_lib.Oracle(s)
    fl = o.type == 0
    o.step(warm)
    t_or = []
    for _ in range(blocks):
        kt = []
        for _ in range(per):
            o.step(10)
            kt.append((o.v[fl] ** 2).mean())
        t_or.append(np.mean(kt))

    sim = dpd.Simulation(s, graph=True)
    sim.step(warm)
    t_gpu = []
    for _ in range(blocks):
        acc = None
        for _ in range(per):
            sim.step(10)
            p = sim.profile(axis=2, nbins=1)
            acc = p if acc is None else acc + p
        a = acc.cpu().numpy()[0]
        t_gpu.append(a[4] / (3.0 * a[0]))
    c = sim.counters()
    sim.close()
    se = lambda x: np.std(x, ddof=1) / np.sqrt(len(x))
    say("T gpu %.4f +- %.4f  oracle %.4f +- %.4f" % (np.mean(t_gpu), se(t_gpu), np.mean(t_or), se(t_or)))
    assert c["unstable"] == 0
    tol = 3 * np.hypot(se(t_gpu), se(t_or)) + 0.01
    assert abs(np.mean(t_gpu) - np.mean(t_or)) < tol


def test_adjoint_refuses_the_force(dpd):
    from paper_1807_09896_amd.adjoint import Window
    sim = dpd.Simulation(_with_sph(workloads.tiny_slab_system()))
    w = Window(sim, steps=4, ckpt=2)
    with pytest.raises(dpd.DPDError):
        w.run()
    sim.close()

"""Small flames whose steps run in one launch, a workgroup per flame: against
the FP64 oracle on every kind of grid the kernel has, and bit for bit over
splits of a run, graphs, ensembles, the allocation-free call and (where both
axes have a product grid) the two-kernel step."""

import ctypes

import numpy as np
import pytest

import oracle
import synth
from flame_testlib import oracle_trajectory, rel_l2

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

GRIDS = [(16, 16), (16, 32), (32, 16), (16, 512), (32, 64), (64, 32), (32, 256), (64, 64), (64, 128), (128, 16),
         (128, 32), (128, 64), (128, 128), (256, 64), (512, 32), (1024, 16)]


def workload(n1, n2, amp=0.1):
    return synth.Workload(f"r{n1}x{n2}", n1, n2, 1, 0.2, "all", amp, -1.0, 5 * n1 + n2, t0=5.0)


def make(w, **kw):
    from paper_0911_2889_amd import FlameSim
    return FlameSim(w.n1, w.n2, gamma=w.gamma, theta_pi=w.theta_pi, t0=w.t0, dt=w.dt, **kw)


@pytest.mark.parametrize("n1,n2", GRIDS)
@pytest.mark.parametrize("kind", ["euler", "rk2", "forced", "forced rk2"])
def test_resident_steps_match_oracle(n1, n2, kind):
    w = workload(n1, n2)
    half = synth.workload_spectrum(w)
    integrator = "rk2" if "rk2" in kind else "euler"
    kw = dict(gamma=w.gamma, theta_pi=w.theta_pi, t0=w.t0, dt=w.dt, integrator=integrator)
    sim = make(w, integrator=1 if integrator == "rk2" else 0)
    if "forced" in kind:
        fh = synth.forcing_spectrum(w, amp=1e-2)
        kw["forcing"] = oracle.half_to_full(fh.astype(np.complex128), n1, n2)
        sim.set_forcing(fh)
    refs = oracle_trajectory(half, oracle.Params(n1, n2, **kw), [1, 20])
    sim.set_spectrum(half)
    sim.step(1)
    # the bounds of the two-kernel step's tests
    assert rel_l2(sim.spectrum().cpu().numpy(), refs[1]) < 1e-6
    sim.step(19)
    assert rel_l2(sim.spectrum().cpu().numpy(), refs[20]) < 1e-5
    assert sim.step_index == 20 and sim.diagnostics()["finite"]


@pytest.mark.parametrize("n1,n2", [(16, 16), (64, 128), (128, 128), (1024, 16)])
@pytest.mark.parametrize("integrator", [0, 1])
def test_resident_steps_do_not_depend_on_how_they_are_launched(n1, n2, integrator):
    """130 steps: more than two of the chunks in which the kernel forms its scalars."""
    from paper_0911_2889_amd import FlameEnsemble, native
    w = workload(n1, n2, amp=1e-3)
    half = synth.workload_spectrum(w)
    whole = make(w, integrator=integrator)
    whole.set_spectrum(half)
    whole.step(130)
    ref = whole.spectrum()
    parts = make(w, integrator=integrator)
    parts.set_spectrum(half)
    for k in (1, 63, 2, 64):
        parts.step(k)
    assert torch.equal(parts.spectrum(), ref)
    graph = make(w, integrator=integrator)
    graph.set_graph_steps(40)
    graph.set_spectrum(half)
    for _ in range(3):
        graph.step(40)
        graph.diagnostics()
    graph.step(10)
    assert torch.equal(graph.spectrum(), ref)
    kw = dict(gamma=w.gamma, theta_pi=w.theta_pi, t0=w.t0, dt=w.dt, integrator=integrator)
    ens = FlameEnsemble([dict(n1=n1, n2=n2, **kw)] * 3 + [dict(n1=256, n2=512, **kw)])
    for f in range(3):
        ens.set_spectrum(half, flame=f)
    ens.step(130)
    assert all(torch.equal(ens.spectrum(f), ref) for f in range(3))
    if integrator == 0:
        solo = make(w)
        solo.set_spectrum(half)
        lib = native.load()
        native.check(lib.flame_step_noalloc(ctypes.byref(solo.descs[0]), ctypes.c_void_p(solo.states[0].data_ptr()), 0,
                                            130, ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)))
        assert torch.equal(solo.spectrum(), ref)
    if n1 >= 128 and n2 >= 64:
        two = make(w, integrator=integrator)
        two.set_points_per_thread(n1, n2, 12, 12)
        two.set_spectrum(half)
        two.step(130)
        assert torch.equal(two.spectrum(), ref)


def test_resident_radius_table_and_switches():
    """A tabulated radius, and leaving and re-entering the one-launch step in mid-run."""
    w = workload(64, 128)
    half = synth.workload_spectrum(w)
    t = w.t0 + w.dt * np.arange(42)
    tab = np.stack([t[:-1], np.log1p(w.dt / t[:-1]), w.dt / (t[:-1] * t[1:])], axis=1)  # r0 = t, as a table
    a, b = make(w), make(w, r0_law=1)
    b.set_r0_table(torch.from_numpy(tab).cuda())
    for sim in (a, b):
        sim.set_spectrum(half)
    a.step(20)
    b.step(8)
    b.set_points_per_thread(64, 128, 8, 8)
    b.step(4)
    b.set_points_per_thread(64, 128, 16, 16)
    b.step(8)
    assert rel_l2(b.spectrum().cpu().numpy(), a.spectrum().cpu().numpy()) < 2e-6
    ref = oracle_trajectory(half, oracle.Params(64, 128, gamma=w.gamma, theta_pi=w.theta_pi, t0=w.t0, dt=w.dt), [20])[20]
    assert rel_l2(a.spectrum().cpu().numpy(), ref) < 1e-5

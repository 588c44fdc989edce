"""The step and its adjoint on the paper's N1 x N2 grid (the product grid
disabled), against the FP64 oracle, at the shortest and longest rows of each
plan; with 12 row points per thread the grid has 3 N2/4 phi points."""

import numpy as np
import pytest

import oracle
import synth
from flame_testlib import oracle_trajectory, rel_l2
from test_gpu_adjoint import from_internal, make, spectrum, to_internal

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

GRIDS = [(64, 64), (16, 256), (128, 64), (128, 128), (256, 512), (32, 2048), (128, 4096), (64, 8192), (32, 16384)]


@pytest.mark.parametrize("n1,n2", GRIDS)
@pytest.mark.parametrize("integrator", [0, 1])
def test_steps_on_the_full_grid_match_the_oracle(n1, n2, integrator):
    from paper_0911_2889_amd import FlameSim
    w = synth.Workload(f"f{n1}x{n2}", n1, n2, 1, 0.2, "all", 0.1, -1.0, n1 + 3 * n2, t0=5.0)
    half = synth.workload_spectrum(w)
    p = oracle.Params(n1, n2, gamma=w.gamma, theta_pi=w.theta_pi, t0=w.t0, dt=w.dt,
                      integrator="rk2" if integrator else "euler")
    ref = oracle_trajectory(half, p, [3])[3]
    outs = {}
    for rp in (16, 8, 12):
        if rp == 8 and n2 > 8192:
            continue  # refused there
        sim = FlameSim(n1, n2, gamma=w.gamma, theta_pi=w.theta_pi, t0=w.t0, dt=w.dt, integrator=integrator)
        sim.set_product_grid(n1, n2, False)
        sim.set_points_per_thread(n1, n2, 16, rp)
        sim.set_spectrum(half)
        sim.step(1)
        sim.set_graph_steps(2)
        sim.step(2)
        outs[rp] = sim.spectrum().cpu().numpy()
        assert rel_l2(outs[rp], ref) < 2e-6, rp  # the bound of the product grids' test
    assert not np.array_equal(outs[16], outs[12])  # transforms of other lengths


@pytest.mark.parametrize("n1,n2", GRIDS)
@pytest.mark.parametrize("rp", [16, 12])
def test_adjoint_step_on_the_full_grid(n1, n2, rp):
    t0, dt, n = 5.0, 0.2, 3
    state, lam = spectrum(n1, n2, 31 + n1, 0.3), spectrum(n1, n2, 32 + n2, 1.0)
    sim = make(n1, n2, t0, dt)
    sim.set_product_grid(n1, n2, False)
    sim.set_points_per_thread(n1, n2, 16, rp)
    li, st = to_internal(lam, n1, n2), to_internal(state, n1, n2)
    sim.adjoint_step(n, st, li, li)
    got = from_internal(li, n1, n2)
    p = oracle.Params(n1, n2, t0=t0, dt=dt)
    sf = oracle.half_to_full(state.astype(np.complex128), n1, n2)
    lf = oracle.half_to_full(lam.astype(np.complex128), n1, n2)
    ref = oracle.full_to_half(oracle.step_adjoint(sf, lf, p, n), n1, n2)
    # five transforms of at most 2^14 points at 2.6e-7 each
    assert rel_l2(got, ref) < 2e-6


@pytest.mark.parametrize("n1,n2", [(64, 64), (16, 1024), (64, 8192)])
def test_adjoint_step_on_short_columns_by_default(n1, n2):
    """N1 rows and 3 N2/4 phi points, the default where n1 < 128."""
    t0, dt, n = 5.0, 0.2, 3
    state, lam = spectrum(n1, n2, 31 + n1, 0.3), spectrum(n1, n2, 32 + n2, 1.0)
    sim = make(n1, n2, t0, dt)
    li, st = to_internal(lam, n1, n2), to_internal(state, n1, n2)
    sim.adjoint_step(n, st, li, li)
    p = oracle.Params(n1, n2, t0=t0, dt=dt)
    sf = oracle.half_to_full(state.astype(np.complex128), n1, n2)
    lf = oracle.half_to_full(lam.astype(np.complex128), n1, n2)
    ref = oracle.full_to_half(oracle.step_adjoint(sf, lf, p, n), n1, n2)
    assert rel_l2(from_internal(li, n1, n2), ref) < 2e-6

"""The product-grid step kernels: the bodies for many and for few transforms
give the same bits, on grids at the edges of every length's plan and on both
sides of the rule that chooses between them, and match the FP64 oracle."""

import numpy as np
import pytest

import oracle
import synth
from flame_testlib import oracle_trajectory, rel_l2

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n1,n2", [(128, 64), (128, 16), (128, 128), (256, 2048), (128, 4096), (512, 64), (1024, 128),
                                   (2048, 64), (4096, 64), (8192, 64), (64, 64), (32, 512), (16, 8192), (1024, 2048)])
@pytest.mark.parametrize("integrator", [0, 1])
def test_bodies_agree_bit_for_bit_and_with_the_oracle(n1, n2, integrator):
    from paper_0911_2889_amd import FlameSim
    w = synth.Workload(f"m{n1}x{n2}", n1, n2, 1, 0.2, "all", 0.1, -1.0, n1 + 3 * n2, t0=5.0)
    half = synth.workload_spectrum(w)
    outs = {}
    for cp, rp in ((16, 16), (8, 8), (12, 12)):
        if (cp == 12 and n1 < 128) or (rp == 12 and n2 < 64):
            continue  # refused there: no product grid
        sim = FlameSim(n1, n2, gamma=w.gamma, theta_pi=w.theta_pi, t0=w.t0, dt=w.dt, integrator=integrator)
        sim.set_points_per_thread(n1, n2, cp, rp)
        sim.set_spectrum(half)
        sim.step(3)
        outs[cp] = sim.spectrum().cpu().numpy()
    if n1 * n2 <= 1 << 19:
        p = oracle.Params(n1, n2, gamma=w.gamma, theta_pi=w.theta_pi, t0=w.t0, dt=w.dt,
                          integrator="rk2" if integrator else "euler")
        ref = oracle_trajectory(half, p, [3])[3]
        for cp in outs:
            assert rel_l2(outs[cp], ref) < 2e-6, cp
    if n1 >= 128 and n2 >= 64:  # below, the points per thread select other transforms
        for cp in outs:
            assert np.array_equal(outs[cp], outs[16]), cp


def test_solo_and_many_agree_across_the_rule():
    """One 256x512 flame runs the bodies for few transforms, thirty-three of them the others."""
    from paper_0911_2889_amd import FlameEnsemble, FlameSim
    w = synth.Workload("r", 256, 512, 1, 0.2, "all", 0.1, -1.0, 9, t0=5.0)
    half = synth.workload_spectrum(w)
    kw = dict(n1=256, n2=512, gamma=w.gamma, t0=w.t0, dt=w.dt)
    solo = FlameSim(**kw)
    solo.set_spectrum(half)
    solo.step(4)
    many = FlameEnsemble([kw] * 33)
    for f in range(33):
        many.set_spectrum(half, flame=f)
    many.step(4)
    for f in (0, 16, 32):
        assert torch.equal(many.spectrum(f), solo.spectrum())

"""The averages on both sides of the rule that puts their row transforms side by
side, for short rows: grids of which the rule for long rows would take either side."""

import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n1,n2", [(4096, 32), (16384, 32), (2048, 256), (4096, 256), (4096, 512), (16384, 128),
                                   (1024, 1024), (2048, 1024)])
def test_averages_of_short_rows(n1, n2):
    from paper_0911_2889_amd import FlameSim
    w = synth.Workload(f"a{n1}x{n2}", n1, n2, 1, 0.2, "all", 0.1, -1.0, n1 + 7 * n2, t0=5.0)
    half = synth.workload_spectrum(w)
    sim = FlameSim(n1, n2, gamma=0.8, theta_pi=0.2, t0=5.0, dt=0.1)
    sim.set_spectrum(half)
    p = oracle.Params(n1, n2, gamma=0.8, theta_pi=0.2, t0=5.0, dt=0.1)
    full = oracle.symmetrise(oracle.half_to_full(half.astype(np.complex128), n1, n2))
    r, v, a = oracle.diagnostics(full, p, 0)
    got = sim.diagnostics()
    # the bounds of the averages' other test
    assert got["finite"]
    assert abs(got["mean_radius"] - r) < 1e-9 * abs(r)
    assert abs(got["velocity"] - v) < 2e-5 * abs(v)
    assert abs(got["area_excess"] - a) < 2e-5 * abs(a)
    assert sim.diagnostics() == got

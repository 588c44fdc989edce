"""The kernels on the physical grid: the averages of a state in one launch
(their partial sums meet in the workgroup that finishes last) and the half
spectrum to and from the state layout in tiles."""

import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# the smallest grids; one workgroup and fewer than there are counters; both sides of the rule
# for transforms side by side (N1 N2 = 2^21, N2 = 2048); the tiles of the spectrum's copy cut
# at both ends; the longest rows
GRIDS = [(16, 16), (16, 512), (32, 64), (64, 32), (256, 512), (2048, 64), (1024, 2048), (2048, 2048), (512, 4096),
         (64, 8192), (32, 16384)]


def make(n1, n2, **kw):
    from paper_0911_2889_amd import FlameSim
    return FlameSim(n1, n2, gamma=0.8, theta_pi=0.2, t0=5.0, dt=0.1, **kw)


@pytest.mark.parametrize("n1,n2", GRIDS)
@pytest.mark.parametrize("scale", [1.0, 1e15])
def test_averages_match_the_oracle_each_time(n1, n2, scale):
    """At scale 1e15 the squared gradients pass 1e30, where the area excess
    takes its plain form; a state that is not finite in between is flagged and
    leaves nothing behind."""
    w = synth.Workload(f"p{n1}x{n2}", n1, n2, 1, 0.2, "all", 0.1, -1.0, n1 + 7 * n2, t0=5.0)
    half = (synth.workload_spectrum(w) * scale).astype(np.complex64)
    sim = make(n1, n2)
    sim.set_spectrum(half)
    p = oracle.Params(n1, n2, gamma=0.8, theta_pi=0.2, t0=5.0, dt=0.1)
    full = oracle.symmetrise(oracle.half_to_full(half.astype(np.complex128), n1, n2))
    r, v, a = oracle.diagnostics(full, p, 0)
    first = sim.diagnostics()
    assert first["finite"]
    # the bounds of the averages' other test
    assert abs(first["mean_radius"] - r) < 1e-9 * abs(r)
    assert abs(first["velocity"] - v) < 2e-5 * abs(v)
    assert abs(first["area_excess"] - a) < 2e-5 * abs(a)
    bad = half.copy()
    bad[-1, -1] = np.nan
    sim.set_spectrum(bad)
    assert not sim.diagnostics()["finite"]
    sim.set_spectrum(half)
    for _ in range(3):
        assert sim.diagnostics() == first


@pytest.mark.parametrize("n1,n2", GRIDS)
def test_spectrum_goes_in_and_out_unchanged(n1, n2):
    rng = np.random.default_rng(n1 + n2)
    shape = (n1 // 2 - 1, n2 // 4)
    half = (rng.standard_normal(shape) + 1j * rng.standard_normal(shape)).astype(np.complex64)
    k1 = n1 // 4 - 1
    half[:k1, 0] = np.conj(half[k1 + 1:, 0][::-1])
    half[k1, 0] = half[k1, 0].real
    sim = make(n1, n2)
    given = half.copy()
    given[:k1, 0] = 7.0  # k2 = 0: the k1 < 0 half follows from the other one
    given[k1, 0] += 3.0j
    sim.set_spectrum(given)
    assert np.array_equal(sim.spectrum().cpu().numpy(), half)


@pytest.mark.parametrize("n1,n2", GRIDS)
@pytest.mark.parametrize("product", [True, False])
def test_projection_leaves_a_state_that_steps(n1, n2, product):
    """The column transforms after a projection on the product rows are formed
    at the next step, on N1 rows at once; the averages need N1 rows of both."""
    phi = synth.physical_noise(n1, n2, seed=n1 + n2, kind="uniform", scale=1e-3)
    one, two = make(n1, n2), make(n1, n2)
    for s in (one, two):
        if n1 >= 128:  # shorter columns have no product grid
            s.set_product_grid(n1, n2, product)
    one.set_phi(phi)
    two.set_spectrum(one.spectrum())
    assert one.diagnostics() == two.diagnostics()
    one.set_phi(phi)
    for s in (one, two):
        s.step(2)
    assert torch.equal(one.states[0], two.states[0])

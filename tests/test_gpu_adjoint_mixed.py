"""The adjoint step's product-grid kernels against the FP64 oracle: every
length's plan, side-by-side and one-after-another transforms (the larger grids
and the long axes), and the grids where only one axis has a product grid."""

import numpy as np
import pytest

import oracle
from flame_testlib import rel_l2
from test_gpu_adjoint import from_internal, make, spectrum, to_internal

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n1,n2", [(128, 16), (128, 128), (64, 64), (16, 1024), (512, 256), (128, 4096), (1024, 2048),
                                   (4096, 64), (128, 8192), (8192, 64)])
@pytest.mark.parametrize("product", [True, False])
def test_adjoint_step_on_product_grids(n1, n2, product):
    if not product and n1 < 128:
        pytest.skip("no theta product grid to switch off")
    t0, dt, n = 5.0, 0.2, 3
    state, lam = spectrum(n1, n2, 31 + n1, 0.3), spectrum(n1, n2, 32 + n2, 1.0)
    sim = make(n1, n2, t0, dt)
    sim.set_product_grid(n1, n2, product and n1 >= 128)
    li = to_internal(lam, n1, n2)
    st = to_internal(state, n1, n2)
    sim.adjoint_step(n, st, li, li)
    got = from_internal(li, n1, n2)
    p = oracle.Params(n1, n2, t0=t0, dt=dt)
    sf = oracle.half_to_full(state.astype(np.complex128), n1, n2)
    lf = oracle.half_to_full(lam.astype(np.complex128), n1, n2)
    ref = oracle.full_to_half(oracle.step_adjoint(sf, lf, p, n), n1, n2)
    # five transforms of at most 2^13 points at 2.6e-7 (the mixed transforms' bound) each
    assert rel_l2(got, ref) < 2e-6

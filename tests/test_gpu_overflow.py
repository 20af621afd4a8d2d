"""Values past the largest float64: the Laplacian divides by h^2 through the
reciprocal of it, and a quotient that overflows has to be the infinity that
the division gives.

Oracle: numpy.  The inputs are powers of two, so every sum is exact and every
quotient either exact or infinite: no tolerance."""
import numpy as np
import pytest

from paper_2501_15314_amd import workloads as wl

from .conftest import gpu_available
from .test_gpu_cycle import F, N, P, _stencil

pytestmark = pytest.mark.gpu

if gpu_available():
    from paper_2501_15314_amd.sim import Sim


@pytest.mark.parametrize("bc", [(P, P, P), (N, P, F)])
@pytest.mark.parametrize("scale", [1015, 1016, 1020])  # largest sums 12 x 2^scale, over h^2 = 2^-8
def test_laplacian_past_the_largest_value(scale, bc):
    n, h = (16, 20, 24), 1.0 / 16
    cfg = wl.Config(n=n, length=tuple(x * h for x in n), bc=bc, nu=0.02, dt=0.01, precond=wl.PRECOND_FASTDIAG_EXACT)
    x = np.random.default_rng(scale).choice([-1.0, 0.0, 1.0], n) * 2.0 ** scale
    sim = Sim(cfg, 0)
    got = sim.apply("laplacian", x).cpu().numpy()
    sim.close()
    nb, nn = _stencil(x, bc)
    with np.errstate(over="ignore"):
        ref = (nn * x - nb) / (h * h)
    assert np.isinf(ref).any() == (scale > 1014) and np.isfinite(ref).any()
    assert np.array_equal(got, ref)

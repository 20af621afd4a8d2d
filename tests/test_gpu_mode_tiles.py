"""The float64 mode products at the edges of their tiles (32 entries of either
parity x 64 lines, summation steps of 8): half sizes 8 to 66, one below, at
and above a tile, and line counts that leave partial tiles.  Oracle: the
FFT/DCT pseudo-inverse.  Tolerance: six products of at most n / 2 = 66 terms
and the oracle's transforms round at about 1e-15 relative each, against
1e-12."""
import numpy as np
import pytest

from oracle import mac as omac
from oracle import poisson as opoisson
from paper_2501_15314_amd import workloads as wl

from .conftest import gpu_available
from .gpu_helpers import rel

pytestmark = pytest.mark.gpu

if gpu_available():
    from paper_2501_15314_amd.sim import Sim


@pytest.mark.parametrize("bc", [(0, 0, 0), (1, 2, 1), (0, 1, 0)])
@pytest.mark.parametrize("n", [(16, 60, 64), (64, 68, 16), (68, 16, 60), (20, 64, 132), (132, 20, 28)])
def test_mode_products_at_tile_edges(n, bc):
    cfg = wl.Config(n=n, length=tuple(x / 32.0 for x in n), bc=bc, precond=wl.PRECOND_FASTDIAG_EXACT)
    sim = Sim(cfg, 1)
    b = np.random.default_rng(sum(n)).standard_normal(n)
    z = sim.apply("precond", b).cpu().numpy()
    assert rel(z, opoisson.solve_laplacian(omac.Grid(cfg.n, cfg.h, cfg.bc), b)) < 1e-12
    sim.close()

"""March tiles one pair of cells wide: rows of 4 cells on a marched multigrid
level (their sweeps, restriction and first sweeps), and rows whose quarter is a
prime above 64 in chunks of several planes.

Oracles and tolerances: the array cycle of test_gpu_cycle and the explicit
sparse operators, as there and in test_gpu_march_shapes."""
import numpy as np
import pytest

from oracle import mac as omac
from paper_2501_15314_amd import workloads as wl

from .conftest import gpu_available
from .gpu_helpers import make_sim, mg_tile_cells, rel
from .test_gpu_cycle import F, N, P, _cycle

pytestmark = pytest.mark.gpu

if gpu_available():
    from paper_2501_15314_amd.sim import Sim


@pytest.mark.parametrize("precision", [wl.PREC_FP64, wl.PREC_FP32MG])
@pytest.mark.parametrize("sweeps", [(2, 1), (1, 2)])
@pytest.mark.parametrize("bc", [(P, P, P), (N, P, F), (F, N, P)])
def test_cycle_with_rows_of_four_cells(bc, sweeps, precision):
    # 64 x 32 x 4 cells above 32 x 16 x 2: too many for the two-level workgroup
    n, h, coarsest = (256, 128, 16), 1.0 / 32, 32
    cfg = wl.Config(n=n, length=tuple(x * h for x in n), bc=bc, nu=0.02, dt=0.005, precision=precision, mg_coarsest=coarsest,
                    mg_pre=sweeps[0], mg_post=sweeps[1], mg_coarse_sweeps=0)
    with mg_tile_cells(0):
        sim = Sim(cfg, 1)
    b = np.random.default_rng(sweeps[0]).standard_normal(n)
    b -= b.mean()
    z = sim.apply("precond", b).cpu().numpy()
    sim.close()
    ref = _cycle(b, h, bc, coarsest, *sweeps)
    assert rel(z - z.mean(), ref - ref.mean()) < (1e-12 if precision == wl.PREC_FP64 else 1e-4)


@pytest.mark.parametrize("bc", [(P, P, P), (N, P, F), (F, N, N)])
@pytest.mark.parametrize("n", [(20, 24, 284), (20, 64, 268), (16, 76, 292)])  # 24, 32 (two tiles) and 76 rows
def test_stencils_in_chunks_of_eight_planes(n, bc):
    h = 1.0 / 16
    cfg = wl.Config(n=n, length=tuple(x * h for x in n), bc=bc, nu=0.02, dt=0.01, precision=wl.PREC_FP64,
                    precond=wl.PRECOND_FASTDIAG_EXACT, helm_rtol=1e-12)
    sim = make_sim(cfg, 0, "full")
    g = omac.Grid(n, h, bc)
    rng = np.random.default_rng(71)
    x = rng.standard_normal(n)
    assert rel(sim.apply("laplacian", x).cpu().numpy().ravel(), omac.laplacian(g) @ x.ravel()) < 1e-13
    r = rng.standard_normal((3,) + n) * g.face_dof_mask()
    u = sim.apply("helm_solve", r).cpu().numpy()
    assert rel(omac.helmholtz(g, cfg.nu, cfg.dt) @ u.ravel(), r.ravel()) < 2.0 * cfg.helm_rtol
    sim.close()

"""Momentum sweeps and residuals whose workgroups march over two planes where
those of one field take one.  Oracle: the explicit sparse operator, at the
solve's own target."""
import numpy as np
import pytest

from oracle import mac as omac
from paper_2501_15314_amd import workloads as wl

from .conftest import gpu_available
from .gpu_helpers import CHUNKS, make_sim, rel

pytestmark = pytest.mark.gpu

P, N, F = wl.BC_PERIODIC, wl.BC_NOSLIP, wl.BC_FREESLIP


@pytest.mark.parametrize("chunks", CHUNKS)
@pytest.mark.parametrize("precision", [wl.PREC_FP64, wl.PREC_FP32MG])
@pytest.mark.parametrize("n,bc", [((48, 96, 128), (N, P, F)), ((48, 96, 128), (P, F, N)), ((64, 80, 80), (P, P, P)), ((32, 64, 160), (F, N, P))])
def test_momentum_solve_in_chunks_of_two_planes(n, bc, precision, chunks):
    h = 1.0 / 64
    cfg = wl.Config(n=n, length=tuple(x * h for x in n), bc=bc, nu=0.02, dt=0.01, precision=precision,
                    precond=wl.PRECOND_FASTDIAG_EXACT if precision == wl.PREC_FP64 else wl.PRECOND_FASTDIAG,
                    helm_rtol=1e-12 if precision == wl.PREC_FP64 else 1e-10)
    sim = make_sim(cfg, 0, chunks)
    g = omac.Grid(n, h, bc)
    r = np.random.default_rng(n[0]).standard_normal((3,) + n) * g.face_dof_mask()
    u = sim.apply("helm_solve", r).cpu().numpy()
    sim.close()
    assert rel(omac.helmholtz(g, cfg.nu, cfg.dt) @ u.ravel(), r.ravel()) < 2.0 * cfg.helm_rtol

"""The list kernels of the coupling term (k_interp and k_band of
kernels_ib.hip), which serve the float32 form and the bf16 preconditioner,
where their work split changes: chunks of 32 and 64 points, tiles cut into
several workgroups, few tiles (staged beside the accumulation) and many.

Oracle: the explicit sparse matrices of oracle.schur.  Tolerance of the
float64 products: a cell sums at most 600 points x 64 nodes, about 1200
roundings in a row plus the cancellation of the divergence (a factor of about
10): 1200 x 10 x 1.1e-16 < 2e-12.  The float32 form solves to its bar of 1e-8."""
import numpy as np
import pytest

from oracle import delta as odelta
from oracle import mac as omac
from oracle import schur as oschur
from paper_2501_15314_amd import workloads as wl

from .conftest import gpu_available
from .gpu_helpers import rel

pytestmark = pytest.mark.gpu

if gpu_available():
    from paper_2501_15314_amd.sim import Sim

P3 = (wl.BC_PERIODIC,) * 3


def _sim(n, X, delta, precision, points):
    h = 1.0 / 16
    cfg = wl.Config(n=n, length=tuple(x * h for x in n), bc=P3, nu=0.02, dt=0.005, delta=delta, lump_c=0.4 + 0.1 * points,
                    precision=precision, precond=wl.PRECOND_FASTDIAG if precision == wl.PREC_FP64 else wl.PRECOND_VCYCLE,
                    krylov_rtol=1e-12 if precision == wl.PREC_FP64 else 1e-9, mg_coarsest=16)
    sim = Sim(cfg, len(X))
    sim.set_bodies([wl.Body(center=np.zeros(3), vel=np.zeros(3), omega=np.zeros(3), radius=1.0, n_points=len(X))], X)
    g = omac.Grid(n, h, P3)
    return sim, oschur.SchurSystem(g, odelta.regularization_matrix(g, sim.get_points()[0].cpu().numpy(), delta), cfg.lump_c)


def _one_tile(points, corner, rng, h=1.0 / 16):
    """All points inside one tile -- at the grid's corner, moved by a period,
    so that the support wraps, or in the interior -- and two elsewhere."""
    lo = np.array([-16, 0, 32] if corner else [8, 8, 12]) * h
    X = lo + rng.uniform(0.0, 4.0, (points, 3)) * h
    return np.concatenate([X, np.array([[8.3, 7.8, 9.1], [9.5, 10.25, 9.0]]) * h])


@pytest.mark.parametrize("delta", [wl.DELTA_PESKIN4, wl.DELTA_ROMA3])
@pytest.mark.parametrize("corner", [False, True])
@pytest.mark.parametrize("points", [1, 31, 32, 33, 64, 65, 129, 256, 257, 600])
def test_list_product_at_the_edges_of_its_chunks(points, corner, delta):
    rng = np.random.default_rng(points)
    sim, S = _sim((16, 24, 32), _one_tile(points, corner, rng), delta, wl.PREC_FP64, points)
    z = rng.standard_normal(S.g.n)
    assert rel(sim.apply("schur", z).cpu().numpy(), S.matvec(z)) < 2e-12
    rf = rng.standard_normal((points + 2, 3))
    assert rel(sim.apply("schur_rhs", np.zeros(S.g.n), rf).cpu().numpy(), S.rhs(np.zeros(S.g.n), rf)) < 2e-12
    sim.close()


@pytest.mark.parametrize("delta", [wl.DELTA_PESKIN4, wl.DELTA_ROMA3])
@pytest.mark.parametrize("points", [33, 257])
def test_float32_list_products_solve_to_their_bar(points, delta):
    rng = np.random.default_rng(points)
    sim, S = _sim((16, 24, 32), _one_tile(points, True, rng), delta, wl.PREC_FP32MG, points)
    rp, rf = rng.standard_normal(S.g.n), rng.standard_normal((points + 2, 3))
    p, phi, _ = sim.solve_schur(rp - rp.mean(), rf)
    p_ref, phi_ref, _, _ = S.solve(rp - rp.mean(), rf)
    assert rel(p.cpu().numpy(), p_ref) < 1e-8
    assert rel(phi.cpu().numpy(), phi_ref) < 1e-8
    sim.close()


@pytest.mark.parametrize("precision", [wl.PREC_FP64, wl.PREC_FP32MG])
def test_more_tiles_than_resident_workgroups(precision):
    # 9000 points scattered over 2048 tiles of 4^3 cells, all of them active
    rng = np.random.default_rng(5)
    n = (32, 64, 64)
    X = rng.uniform(0.0, 1.0, (9000, 3)) * np.array(n) / 16.0
    sim, S = _sim(n, X, wl.DELTA_PESKIN4, precision, 40)
    z, rf = rng.standard_normal(n), rng.standard_normal((len(X), 3))
    if precision == wl.PREC_FP64:
        assert rel(sim.apply("schur", z).cpu().numpy(), S.matvec(z)) < 2e-12
        assert rel(sim.apply("schur_rhs", z, rf).cpu().numpy(), S.rhs(z, rf)) < 2e-12
    else:
        p, phi, _ = sim.solve_schur(z - z.mean(), rf)
        p = p.cpu().numpy()
        # the residual of the solve, by the oracle's matrices
        b = S.rhs(z - z.mean(), rf)
        assert rel(S.matvec(p), b) < 2e-9
    sim.close()

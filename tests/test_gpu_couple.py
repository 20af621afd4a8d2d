"""The coupling term of S~ (kernels_couple.hip) at the point counts where its
work split changes: groups of 16 points per wavefront, at most 64 per
workgroup, tiles cut into several workgroups, and supports that reach the
regions of neighbouring tiles across periodic boundaries.

Oracle: the explicit sparse matrices of oracle.schur.  Tolerances: a cell
sums at most 200 points x 64 nodes in float64, about 400 roundings in a row
plus the cancellation of the divergence (a factor of about 10):
400 x 10 x 1.1e-16 < 1e-12.  The float32 form solves to its bar of 1e-8."""
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


def _case(points, delta, bc, corner, precision=wl.PREC_FP64, n=(16, 20, 24)):
    """All points inside one 4^3-cell tile: the tile at the grid's corner
    (its region wraps; moved by a whole period, so that the positions lie
    outside the grid) or one in its interior, plus two points elsewhere."""
    rng = np.random.default_rng(points)
    h = 1.0 / 16
    lo = np.array([-16, 0, 24] if corner else [8, 8, 12]) * h
    X = lo + rng.uniform(0.0, 4.0, (points, 3)) * h
    X = np.concatenate([X, np.array([[8.3, 7.8, 9.1], [9.5, 10.25, 9.0]]) * h])
    cfg = wl.Config(n=n, length=tuple(x * h for x in n), bc=bc, nu=0.02, dt=0.005, delta=delta, lump_c=0.4 + 0.1 * points,
                    precision=precision, krylov_rtol=1e-12 if precision == wl.PREC_FP64 else 1e-9, mg_coarsest=max(n) // 2)
    body = wl.Body(center=np.zeros(3), vel=np.zeros(3), omega=np.zeros(3), radius=1.0, n_points=len(X))
    if any(b != wl.BC_PERIODIC for b in bc):
        # the wall check uses the sphere that bounds the body's offsets
        body.center = X.mean(axis=0)
    sim = Sim(cfg, len(X))
    sim.set_bodies([body], X - body.center)
    Xd = sim.get_points()[0].cpu().numpy()
    g = omac.Grid(n, h, bc)
    return sim, oschur.SchurSystem(g, odelta.regularization_matrix(g, Xd, delta), cfg.lump_c), rng


P3 = (wl.BC_PERIODIC,) * 3


@pytest.mark.parametrize("delta", [wl.DELTA_PESKIN4, wl.DELTA_ROMA3])
@pytest.mark.parametrize("corner", [False, True])
@pytest.mark.parametrize("points", [1, 15, 16, 17, 63, 64, 65, 128, 129, 200])
def test_product_at_the_edges_of_the_work_split(points, corner, delta):
    sim, S, rng = _case(points, delta, P3, corner)
    z = rng.standard_normal(S.g.n) + 50.0  # an offset far above z's variation: the product must not see it
    got = sim.apply("schur", z).cpu().numpy()
    assert rel(got, S.matvec(z)) < 1e-12
    rf = rng.standard_normal((points + 2, 3))
    got = sim.apply("schur_rhs", np.zeros(S.g.n), rf).cpu().numpy()
    assert rel(got, S.rhs(np.zeros(S.g.n), rf)) < 1e-12
    sim.close()


@pytest.mark.parametrize("delta", [wl.DELTA_PESKIN4, wl.DELTA_ROMA3])
@pytest.mark.parametrize("points", [1, 17, 65, 129])
def test_float32_products_solve_to_their_bar(points, delta):
    sim, S, rng = _case(points, delta, P3, True, precision=wl.PREC_FP32MG)
    rp = rng.standard_normal(S.g.n)
    rf = rng.standard_normal((points + 2, 3))
    p, phi, _ = sim.solve_schur(rp - rp.mean(), rf)
    p_ref, phi_ref, _, _ = S.solve(rp - rp.mean(), rf)
    assert rel(p.cpu().numpy(), p_ref) < 1e-8
    assert rel(phi.cpu().numpy(), phi_ref) < 1e-8
    sim.close()


@pytest.mark.parametrize("bc", [(wl.BC_NOSLIP,) * 3, (wl.BC_FREESLIP, wl.BC_PERIODIC, wl.BC_NOSLIP)])
def test_product_between_walls(bc):
    sim, S, rng = _case(70, wl.DELTA_PESKIN4, bc, False, n=(20, 24, 28))
    z = rng.standard_normal(S.g.n)
    assert rel(sim.apply("schur", z).cpu().numpy(), S.matvec(z)) < 1e-12
    sim.close()


def test_scattered_points_run_in_batches():
    """60000 points scattered over 24576 tiles: more workgroups than the
    region buffer holds at once (16384)."""
    rng = np.random.default_rng(9)
    n, h = (128, 128, 96), 1.0 / 128
    X = rng.uniform(0.0, 1.0, (60000, 3)) * np.array(n) * h
    cfg = wl.Config(n=n, length=tuple(x * h for x in n), bc=P3, nu=0.02, dt=0.005, lump_c=1.0, mg_coarsest=8)
    sim = Sim(cfg, len(X))
    sim.set_bodies([wl.Body(center=np.zeros(3), vel=np.zeros(3), omega=np.zeros(3), radius=1.0, n_points=len(X))], X)
    g = omac.Grid(n, h, P3)
    S = oschur.SchurSystem(g, odelta.regularization_matrix(g, X, cfg.delta), cfg.lump_c)
    z, rf = rng.standard_normal(n), rng.standard_normal((len(X), 3))
    assert rel(sim.apply("schur", z).cpu().numpy(), S.matvec(z)) < 1e-12
    assert rel(sim.apply("schur_rhs", z, rf).cpu().numpy(), S.rhs(z, rf)) < 1e-12
    sim.close()

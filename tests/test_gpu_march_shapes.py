"""Plane-march workgroup shapes on ragged grids: rows whose thread count along
axis 2 (n2 / 4) is 5, 7, 14, 17, 37, 48 and 60, and row counts with few
divisors.  Oracle: the explicit sparse operators, at the tolerances of the
operator parity tests (a handful of float64 roundings per cell) and of the
float64 solves."""
import numpy as np
import pytest

from oracle import mac as omac
from paper_2501_15314_amd import workloads as wl

from .conftest import gpu_available
from .gpu_helpers import oracle_for, rel

pytestmark = pytest.mark.gpu

if gpu_available():
    from paper_2501_15314_amd.sim import Sim

MIXED = (wl.BC_NOSLIP, wl.BC_PERIODIC, wl.BC_FREESLIP)


@pytest.mark.parametrize("precision", [wl.PREC_FP64, wl.PREC_FP32MG])
@pytest.mark.parametrize("n", [(16, 20, 20), (16, 28, 68), (20, 44, 148), (24, 16, 192), (16, 40, 240)])
def test_stencils_on_ragged_rows(n, precision):
    # any axis sizes: a preconditioner without a multigrid hierarchy (its
    # float32 form takes multiples of 8, so it gets the V-cycle-free float64
    # operators through the same kernels where it can)
    if precision == wl.PREC_FP32MG and any(x % 8 for x in n):
        n = tuple(8 * ((x + 7) // 8) for x in n)
    h = 1.0 / 16
    cfg = wl.Config(n=n, length=tuple(x * h for x in n), bc=MIXED, nu=0.02, dt=0.01, precision=precision,
                    precond=wl.PRECOND_FASTDIAG_EXACT if precision == wl.PREC_FP64 else wl.PRECOND_FASTDIAG,
                    helm_rtol=1e-12 if precision == wl.PREC_FP64 else 1e-10)
    sim = Sim(cfg, 0)
    g = omac.Grid(n, h, MIXED)
    rng = np.random.default_rng(n[2])
    x = rng.standard_normal(n)
    assert rel(sim.apply("laplacian", x).cpu().numpy().ravel(), omac.laplacian(g) @ x.ravel()) < 1e-13
    r = rng.standard_normal((3,) + n) * g.face_dof_mask()
    u = sim.apply("helm_solve", r).cpu().numpy()
    assert rel(omac.helmholtz(g, cfg.nu, cfg.dt) @ u.ravel(), r.ravel()) < 2.0 * cfg.helm_rtol
    sim.close()


@pytest.mark.parametrize("n,coarsest", [((40, 48, 56), 14), ((24, 40, 80), 10), ((56, 24, 112), 14)])
def test_solve_on_ragged_multigrid_levels(n, coarsest):
    h = 1.0 / 32
    radius, K = 0.2, 300
    cfg = wl.Config(n=n, length=tuple(x * h for x in n), bc=(wl.BC_PERIODIC,) * 3, nu=0.02, dt=0.005,
                    lump_c=wl.lump_constant(wl.DELTA_PESKIN4, h, K, radius), krylov_rtol=1e-12, mg_coarsest=coarsest)
    body = wl.Body(center=np.array([0.4, 0.5, 1.1]), vel=np.zeros(3), omega=np.zeros(3), radius=radius, n_points=K)
    w = wl.Workload("ragged", cfg, [body], wl.fibonacci_offsets(K, radius), np.zeros((3,) + n))
    _, _, _, S = oracle_for(w)
    sim = Sim(cfg, K)
    sim.set_bodies(w.bodies, w.offsets)
    rp, rf = wl.random_schur_rhs(5, n, K)
    p, phi, _ = sim.solve_schur(rp, rf)
    p_ref, phi_ref, _, _ = S.solve(rp, rf)
    assert rel(p.cpu().numpy(), p_ref) < 1e-10
    assert rel(phi.cpu().numpy(), phi_ref) < 1e-10
    sim.close()


@pytest.mark.parametrize("bc", [MIXED, MIXED[::-1], (wl.BC_PERIODIC,) * 3])
def test_stencils_on_tiles_one_pair_wide(bc):
    # n2 / 4 = 67 is prime and above a wavefront: a workgroup is one pair of
    # cells wide and its threads bring both halo columns of their row
    n, h = (16, 20, 268), 1.0 / 16
    cfg = wl.Config(n=n, length=tuple(x * h for x in n), bc=bc, nu=0.02, dt=0.01, precision=wl.PREC_FP64,
                    precond=wl.PRECOND_FASTDIAG_EXACT, helm_rtol=1e-12)
    sim = Sim(cfg, 0)
    g = omac.Grid(n, h, bc)
    rng = np.random.default_rng(67)
    x = rng.standard_normal(n)
    assert rel(sim.apply("laplacian", x).cpu().numpy().ravel(), omac.laplacian(g) @ x.ravel()) < 1e-13
    r = rng.standard_normal((3,) + n) * g.face_dof_mask()
    u = sim.apply("helm_solve", r).cpu().numpy()
    assert rel(omac.helmholtz(g, cfg.nu, cfg.dt) @ u.ravel(), r.ravel()) < 2.0 * cfg.helm_rtol
    sim.close()


@pytest.mark.parametrize("precision", [wl.PREC_FP64, wl.PREC_FP32MG])
@pytest.mark.parametrize("sweeps", [(2, 1), (1, 1), (2, 2)])
@pytest.mark.parametrize("n,coarsest,bc", [
    ((20, 24, 28), 14, (wl.BC_PERIODIC,) * 3),                           # cut along axes 0 and 2
    ((20, 24, 28), 14, MIXED),
    ((36, 44, 24), 11, MIXED[::-1]),                                      # second level 18 x 22 x 12
    ((36, 44, 24), 11, (wl.BC_PERIODIC,) * 3),
    ((28, 16, 20), 14, (wl.BC_NOSLIP,) * 3),
])
def test_cut_tile_levels_give_the_same_bits(n, coarsest, bc, sweeps, precision):
    # tile levels whose last tiles are cut give every cell the operations of
    # the march kernels in the same order
    from .gpu_helpers import mg_tile_cells
    h = 1.0 / 28
    cfg = wl.Config(n=n, length=tuple(x * h for x in n), bc=bc, nu=0.02, dt=0.005, precision=precision, mg_coarsest=coarsest,
                    mg_pre=sweeps[0], mg_post=sweeps[1], mg_coarse_sweeps=0)
    b = np.random.default_rng(n[0]).standard_normal(n)
    b -= b.mean()
    out = {}
    for cells in (0, None):
        with mg_tile_cells(cells):
            sim = Sim(cfg, 1)
        sim.probe("tile_down")
        out[cells] = sim.apply("precond", b).cpu().numpy(), sim.probe_read("tile_down")[0]
        sim.close()
    assert out[0][1] == 0 and out[None][1] > 0
    assert np.array_equal(out[0][0], out[None][0])


@pytest.mark.parametrize("restart,tiles", [(29, False), (28, True)])
def test_cut_tile_levels_leave_the_static_scratch_its_solves(restart, tiles):
    # 60 x 64 x 64 in float32 with 29 basis vectors fills 63.6 of the 64 MiB of
    # solve_schur_noalloc; a second x for its cut tile levels (1.05 MiB) would
    # pass them, so those levels march.  With 28 there is room.
    n, h, K = (60, 64, 64), 1.0 / 64, 300
    cfg = wl.Config(n=n, length=tuple(x * h for x in n), bc=(wl.BC_PERIODIC,) * 3, nu=0.02, dt=0.005, lump_c=1.0,
                    precision=wl.PREC_FP32MG, mg_coarsest=16, mg_coarse_sweeps=0, krylov_rtol=1e-6, krylov_restart=restart)
    radius = 0.15
    sim = Sim(cfg, K)
    sim.set_bodies([wl.Body(center=np.array([0.4, 0.5, 0.5]), vel=np.zeros(3), omega=np.zeros(3), radius=radius, n_points=K)],
                   wl.fibonacci_offsets(K, radius))
    rp, rf = wl.random_schur_rhs(5, n, K)
    p, f, _ = sim.solve_schur(rp, rf)
    sim.probe("tile_down")
    p1, f1, _ = sim.solve_schur_noalloc(rp, rf)
    assert (sim.probe_read("tile_down")[0] > 0) == tiles
    assert np.array_equal(p.cpu().numpy(), p1.cpu().numpy()) and np.array_equal(f.cpu().numpy(), f1.cpu().numpy())
    sim.close()

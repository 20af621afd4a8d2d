"""The Gram-Schmidt products of FGMRES on grids of fewer entries than the
reduction has threads (workgroups without entries, one partly filled) and of
more.

Oracle: the Arnoldi recurrence itself.  Its residual estimate equals the true
residual of the iterate as long as the basis is orthogonal; classical
Gram-Schmidt loses eps / res^2 of that, below 1e-6 while the residual is above
1e-5, which these few steps leave it at.  A wrong or misplaced product shows
in the estimate at full size."""
import numpy as np
import pytest

from paper_2501_15314_amd import workloads as wl

from .conftest import gpu_available

pytestmark = pytest.mark.gpu

if gpu_available():
    from paper_2501_15314_amd.sim import Sim


@pytest.mark.parametrize("n", [(16, 20, 24), (32, 32, 32), (64, 64, 64), (80, 96, 112)])
@pytest.mark.parametrize("steps", [1, 2, 3, 4])
def test_estimate_is_the_true_residual(n, steps):
    h, rng = 1.0 / 32, np.random.default_rng(steps)
    cfg = wl.Config(n=n, length=tuple(x * h for x in n), bc=(wl.BC_PERIODIC,) * 3, nu=0.02, dt=0.005, lump_c=0.6,
                    precision=wl.PREC_FP64, krylov_restart=steps, krylov_maxit=steps, krylov_rtol=1e-300,
                    mg_coarsest=max(n) // 2 if max(n) < 32 else 14)
    points = rng.uniform(0.2, 0.8, (40, 3)) * np.array(cfg.length)
    sim = Sim(cfg, len(points))
    body = wl.Body(center=np.zeros(3), vel=np.zeros(3), omega=np.zeros(3), radius=1.0, n_points=len(points))
    sim.set_bodies([body], points)
    rp, rf = wl.random_schur_rhs(steps, n, len(points))
    st = sim.solve_schur(rp, rf, allow_notconv=True)[2]
    sim.close()
    est = st.hist[st.nhist - 1]
    print(f"  {n} {steps} steps: estimate {est:.3e} residual {st.rel_res:.3e}")
    assert st.iters == steps
    assert abs(est - st.rel_res) < 1e-6 * st.rel_res

"""The fused passes of a large float32 level (first black and red half sweeps,
last black half sweep and restriction, prolongation and black half sweep) on
row lengths that give their workgroups 8 to 16 rows, an odd number before the
restriction's pairing takes one off among them, and in workgroups of more than
512 threads.

Oracle: the array cycle of test_gpu_cycle, at its tolerance for float32 (a few
hundred roundings of numbers no larger than the result by a factor of ten); and
the separate passes, which give every cell the same operations in the same
order: the same bits."""
import contextlib
import os

import numpy as np
import pytest

from paper_2501_15314_amd import workloads as wl

from .conftest import gpu_available
from .gpu_helpers import rel
from .test_gpu_cycle import F, N, P, _cycle

pytestmark = pytest.mark.gpu

if gpu_available():
    from paper_2501_15314_amd.sim import Sim


def _config(n, bc, coarsest, sweeps):
    h = 1.0 / 128
    return wl.Config(n=n, length=tuple(x * h for x in n), bc=bc, nu=0.02, dt=0.005, precision=wl.PREC_FP32MG, mg_coarsest=coarsest,
                     mg_pre=sweeps[0], mg_post=sweeps[1], mg_coarse_sweeps=0)


def _precond(cfg, b):
    sim = Sim(cfg, 1)
    sim.probe("smooth")
    z, half_sweeps = sim.apply("precond", b).cpu().numpy(), sim.probe_read("smooth")[0]  # launched by themselves
    sim.close()
    return z, half_sweeps


@contextlib.contextmanager
def _separate_passes():
    old = os.environ.get("IBSCHUR_MG_FUSED")
    os.environ["IBSCHUR_MG_FUSED"] = "0"
    try:
        yield
    finally:
        if old is None:
            del os.environ["IBSCHUR_MG_FUSED"]
        else:
            os.environ["IBSCHUR_MG_FUSED"] = old


# the caller's float64 right-hand side takes the fused restriction from 192^3
# cells on
@pytest.mark.parametrize("n,coarsest,sweeps,bc", [
    ((192, 176, 224), 14, (2, 1), (P, P, P)),  # 9 rows by threads, 8 with whole pairs
    ((192, 176, 224), 14, (2, 1), (N, P, F)),
    ((176, 192, 224), 14, (3, 2), (F, N, N)),
    ((256, 192, 160), 16, (2, 2), (N, P, F)),  # 12 rows
    ((224, 192, 192), 14, (2, 1), (F, N, N)),  # 10 rows
    ((160, 160, 320), 20, (2, 1), (P, P, P)),  # 8 rows of 80 threads
    ((160, 160, 320), 20, (2, 1), (N, P, F)),
])
def test_cycle_by_row_length(n, coarsest, sweeps, bc):
    b = np.random.default_rng(n[2]).standard_normal(n)
    b -= b.mean()
    cfg = _config(n, bc, coarsest, sweeps)
    z, ref = _precond(cfg, b)[0], _cycle(b, cfg.h, bc, coarsest, *sweeps)
    assert rel(z - z.mean(), ref - ref.mean()) < 1e-4


@pytest.mark.parametrize("n,coarsest,sweeps,saved", [  # saved: half sweeps without a launch of their own, at least
    ((192, 176, 224), 14, (2, 1), 3),
    ((256, 160, 208), 128, (2, 1), 3),  # 9 rows by threads, above one exact coarse solve
    ((224, 224, 176), 112, (2, 1), 3),  # 11 rows
    ((256, 352, 80), 176, (2, 1), 3),   # 16 rows of 20 threads: five wavefronts
    ((256, 192, 160), 16, (3, 2), 3),   # 12 rows
    ((224, 256, 144), 128, (2, 1), 3),  # 14 rows
    ((224, 192, 192), 14, (2, 2), 3),   # 10 rows
    ((256, 256, 128), 16, (2, 1), 3),   # 16 rows
    ((160, 160, 320), 20, (2, 1), 3),
    ((128, 128, 512), 32, (2, 1), 3),   # 8 rows of 128 threads
    ((144, 128, 128), 9, (2, 1), 2),    # all but the restriction's
    ((96, 112, 224), 14, (2, 1), 2),
    ((144, 128, 128), 9, (1, 1), 1),    # only the prolongation's
    ((144, 128, 128), 9, (2, 0), 1),    # only the first one
    ((64, 64, 96), 12, (2, 1), 1),      # levels of at most 128^3 cells: the first one
    ((32, 32, 288), 18, (2, 1), 1),
    ((128, 16, 256), 16, (2, 1), 1),    # a grid of as few rows as a workgroup may wrap
    ((96, 24, 160), 20, (3, 2), 1),
])
@pytest.mark.parametrize("bc", [(P, P, P), (N, P, F), (F, N, N)])
def test_fused_passes_give_the_bits_of_separate_ones(n, coarsest, sweeps, saved, bc):
    b = np.random.default_rng(n[2]).standard_normal(n)
    b -= b.mean()
    cfg = _config(n, bc, coarsest, sweeps)
    z, few = _precond(cfg, b)
    with _separate_passes():
        ref, all_ = _precond(cfg, b)
    assert np.array_equal(z, ref) and all_ - few >= saved


@pytest.mark.parametrize("n,coarsest", [((96, 112, 224), 14), ((80, 96, 320), 20), ((144, 128, 128), 9)])
@pytest.mark.parametrize("bc", [(P, P, P), (N, P, F)])
def test_fused_passes_in_a_solve(n, coarsest, bc):
    # the cycle on the float32 vectors of the Krylov iteration
    K, radius = 600, 0.2
    cfg = _config(n, bc, coarsest, (2, 1))
    cfg.lump_c, cfg.krylov_rtol = wl.lump_constant(cfg.delta, cfg.h, K, radius), 1e-8
    body = wl.Body(center=np.array([0.3, 0.37, 0.6]), vel=np.zeros(3), omega=np.zeros(3), radius=radius, n_points=K)
    rp, rf = wl.random_schur_rhs(3, n, K)

    def solve():
        sim = Sim(cfg, K)
        sim.set_bodies([body], wl.fibonacci_offsets(K, radius))
        p, phi, st = sim.solve_schur(rp, rf)
        sim.close()
        return p.cpu().numpy(), phi.cpu().numpy(), st.iters

    got = solve()
    with _separate_passes():
        ref = solve()
    assert np.array_equal(got[0], ref[0]) and np.array_equal(got[1], ref[1]) and got[2] == ref[2]

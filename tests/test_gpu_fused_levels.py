"""The fused passes of a large float32 level (first black and red half sweeps,
last black half sweep and restriction, prolongation and black half sweep) on
row lengths that give their workgroups 8 to 14 rows, an odd number before the
restriction's pairing takes one off among them, and in workgroups of more than
512 threads.

Oracle: the array cycle of test_gpu_cycle, at its tolerance for float32 (a few
hundred roundings of numbers no larger than the result by a factor of ten)."""
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
    z = sim.apply("precond", b).cpu().numpy()
    sim.close()
    return z


@pytest.mark.parametrize("n,coarsest,sweeps", [
    ((96, 112, 224), 14, (2, 1)),   # 9 rows by threads, 8 with whole pairs
    ((112, 96, 224), 14, (3, 2)),
    ((128, 112, 160), 10, (2, 2)),  # 12 rows
    ((112, 112, 192), 12, (2, 1)),  # 10 rows
    ((80, 96, 320), 20, (2, 1)),    # 8 rows of 80 threads
])
@pytest.mark.parametrize("bc", [(P, P, P), (N, P, F), (F, N, N)])
def test_cycle_by_row_length(n, coarsest, sweeps, bc):
    b = np.random.default_rng(n[2]).standard_normal(n)
    b -= b.mean()
    cfg = _config(n, bc, coarsest, sweeps)
    z, ref = _precond(cfg, b), _cycle(b, cfg.h, bc, coarsest, *sweeps)
    assert rel(z - z.mean(), ref - ref.mean()) < 1e-4

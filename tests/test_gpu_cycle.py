"""The V-cycle against a numpy one, on hierarchies that reach every variant of
its small levels: tile levels whole and cut, the two-level workgroup with half
and whole quads, with at most 512 threads and with more, and the coarse solve
by itself.

Oracle: the same cycle written with arrays (red-black Gauss-Seidel, the average
of the eight children, trilinear prolongation, a dense solve on the coarsest
grid).  A value passes through a few hundred roundings of numbers no
larger than itself by a factor of about ten: 1e-12 in float64, 1e-4 in
float32."""
import numpy as np
import pytest

from oracle import mac as omac
from paper_2501_15314_amd import workloads as wl

from .conftest import gpu_available
from .gpu_helpers import mg_tile_cells, rel

pytestmark = pytest.mark.gpu

if gpu_available():
    from paper_2501_15314_amd.sim import Sim


def _shift(x, a, s, periodic):
    y = np.roll(x, -s, a)
    if not periodic:
        idx = [slice(None)] * 3
        idx[a] = -1 if s > 0 else 0
        y[tuple(idx)] = 0.0
    return y


def _stencil(x, bc):
    nb, nn = np.zeros_like(x), np.zeros_like(x)
    for a in range(3):
        for s in (-1, 1):
            p = bc[a] == wl.BC_PERIODIC
            nb += _shift(x, a, s, p)
            nn += _shift(np.ones_like(x), a, s, p)
    return nb, nn


def _relax(x, b, h, bc, colour):
    i, j, k = np.indices(x.shape)
    nb, nn = _stencil(x, bc)
    return np.where((i + j + k) % 2 == colour, (h * h * b + nb) / nn, x)


def _interp(c, bc):
    for a in range(3):
        p = bc[a] == wl.BC_PERIODIC
        lo, hi = np.roll(c, 1, a), np.roll(c, -1, a)
        if not p:
            for y, e in ((lo, 0), (hi, -1)):
                idx = [slice(None)] * 3
                idx[a] = e
                y[tuple(idx)] = c[tuple(idx)]
        shape = list(c.shape)
        shape[a] *= 2
        c = np.stack([0.75 * c + 0.25 * lo, 0.75 * c + 0.25 * hi], axis=a + 1).reshape(shape)
    return c


def _cycle(b, h, bc, coarsest, pre, post):
    if max(b.shape) <= coarsest:
        L = omac.laplacian(omac.Grid(b.shape, h, bc)).toarray()
        return np.linalg.solve(L + 1.0 / (h * h * b.size), (b - b.mean()).ravel()).reshape(b.shape)  # mean 0
    x = np.zeros_like(b)
    for _ in range(pre):
        for colour in (0, 1):
            x = _relax(x, b, h, bc, colour)
    nb, nn = _stencil(x, bc)
    r = b - (nn * x - nb) / (h * h)
    n = [m // 2 for m in b.shape]
    x = x + _interp(_cycle(r.reshape(n[0], 2, n[1], 2, n[2], 2).mean((1, 3, 5)), 2 * h, bc, coarsest, pre, post), bc)
    for _ in range(post):
        for colour in (1, 0):
            x = _relax(x, b, h, bc, colour)
    return x


P, N, F = wl.BC_PERIODIC, wl.BC_NOSLIP, wl.BC_FREESLIP


@pytest.mark.parametrize("precision", [wl.PREC_FP64, wl.PREC_FP32MG])
@pytest.mark.parametrize("n,coarsest,sweeps", [
    ((16, 16, 16), 8, (2, 1)),     # two levels: 512 threads
    ((20, 16, 24), 6, (2, 1)),     # tile level, then 10 x 8 x 12 with half quads
    ((48, 24, 24), 12, (1, 2)),    # 24 x 12 x 12 in the two-level workgroup: 576 threads
    ((64, 64, 16), 16, (2, 1)),    # 32 x 32 x 8 above 16 x 16 x 4
    ((128, 128, 16), 16, (1, 1)),  # 32 x 32 x 4: 1024 threads
    ((24, 36, 28), 18, (2, 2)),    # cut tiles, then a coarse solve of 12 x 18 x 14
    ((16, 16, 16), 8, (2, 0)),     # no sweep after the prolongation
    ((16, 16, 16), 16, (2, 1)),    # the coarse solve by itself
    ((20, 32, 16), 8, (2, 1)),     # marched levels below: rows of 8, 16 and 24 entries
    ((32, 24, 48), 12, (2, 1)),
    ((32, 32, 288), 18, (2, 1)),   # and of 144, in workgroups of 576 threads
])
@pytest.mark.parametrize("bc", [(P, P, P), (N, P, F), (F, N, N)])
@pytest.mark.parametrize("tiles", [None, 0])  # small levels as tiles, or all of them marched
def test_cycle_against_arrays(n, coarsest, sweeps, bc, precision, tiles):
    h = 1.0 / 32
    cfg = wl.Config(n=n, length=tuple(x * h for x in n), bc=bc, nu=0.02, dt=0.005, precision=precision, mg_coarsest=coarsest,
                    mg_pre=sweeps[0], mg_post=sweeps[1], mg_coarse_sweeps=0)
    with mg_tile_cells(tiles):
        sim = Sim(cfg, 1)
    b = np.random.default_rng(n[0] + n[2]).standard_normal(n)
    b -= b.mean()
    z = sim.apply("precond", b).cpu().numpy()
    sim.close()
    ref = _cycle(b, h, bc, coarsest, *sweeps)
    assert rel(z - z.mean(), ref - ref.mean()) < (1e-12 if precision == wl.PREC_FP64 else 1e-4)


@pytest.mark.parametrize("bc", [(P, P, P), (N, P, F), (F, N, N)])
def test_cycle_on_a_large_level(bc):
    # above 128^3 cells the prolongation and the black half sweep run as one
    # pass; the last row tile is cut
    n, h, coarsest = (144, 128, 128), 1.0 / 128, 9
    cfg = wl.Config(n=n, length=tuple(x * h for x in n), bc=bc, nu=0.02, dt=0.005, precision=wl.PREC_FP32MG,
                    mg_coarsest=coarsest, mg_coarse_sweeps=0)
    sim = Sim(cfg, 1)
    b = np.random.default_rng(7).standard_normal(n)
    b -= b.mean()
    z = sim.apply("precond", b).cpu().numpy()
    sim.close()
    ref = _cycle(b, h, bc, coarsest, cfg.mg_pre, cfg.mg_post)
    assert rel(z - z.mean(), ref - ref.mean()) < 1e-4

"""Multigrid level kernels at the sizes where they can go wrong, through the
pressure solve (lm_project) against the oracle's exact solve.

Tolerance: the solve stops at relative residual rtol, so the relative error
is at most kappa rtol, kappa = lambda_max / lambda_min of the operator (times
the density ratio), plus the same bound for rounding at 1e-15. rtol = 1e-11: on the long thin grids below the attainable
residual of either precision lies near 1e-13."""
import math

import numpy as np
import pytest

from oracle import Grid, PoissonSolver, beta_inv_rho
from workloads import tanh_stretched_faces, variable_coefficient_problem
from _cases import rel_l2

pytestmark = pytest.mark.gpu
RTOL = 1e-11
WALLS = [("noslip", "noslip"), ("slip", "slip"), ("noslip", "slip")]
OPEN = [("slip", "slip"), ("inflow", "outflow"), ("periodic", "periodic")]


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _kappa(n, L, bc):
    top, low = 0.0, math.inf
    for d, (q, l) in enumerate(zip(n, L)):
        per = bc is None or bc[d][0] == "periodic"
        ih2 = (q / l) ** 2
        top += 4.0 * ih2
        low = min(low, 4.0 * ih2 * math.sin(math.pi / (q if per else 2 * q)) ** 2)
    return top / low


def _check(n, bc=None, precision="fp64", density=False, nu=2, stretch=0.0, rtol=RTOL):
    from paper_2603_01727_amd import Solver
    L = tuple(1.0 + 0.25 * d for d in range(len(n)))
    bc = None if bc is None else bc[:len(n)]
    rho, b = variable_coefficient_problem(n, L, seed=3 + sum(n), kmax=2, m=6)
    faces = [tanh_stretched_faces(q, stretch, l) for q, l in zip(n, L)] if stretch else None
    g = Grid(n, L, bc=None if bc is None else tuple(bc), faces=faces)
    print("levels", n, bc, precision, "density" if density else "", flush=True)
    want = PoissonSolver(g, beta_inv_rho(g, rho) if density else None).solve(b)[0]
    s = Solver(n, L, bc=bc, Re=10.0, dt=1e-3, precision=precision, poisson_rtol=rtol, poisson_maxit=400,
               mg_nu=nu, variable_coefficient=density, faces=faces)
    got, info = s.project(b, rho=rho if density else None)
    s.close()
    err, tol = rel_l2(got, want), _kappa(n, L, bc) * (4.0 if density else 1.0) * max(stretch, 1.0) ** 4 * (rtol + 1e-15)
    print(err, tol, info, flush=True)
    assert info["relres"] <= rtol
    assert err <= tol


# the one-workgroup cycle and solve: a grid that is its own coarsest level
# (odd sizes; up to 64 cells, and beyond, whose inverse is not held on
# chip), all levels in the first wavefront, a last level of more than 64
# cells, the largest grid, two columns of blocks
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("n", [(7, 9), (27, 31), (9, 7, 5), (13, 9, 8), (16, 16), (20, 12), (30, 22), (64, 64), (4, 64),
                               (8, 8, 8), (20, 12, 14), (16, 16, 16)], ids=str)
@pytest.mark.parametrize("bc", [None, WALLS, OPEN], ids=["periodic", "walls", "open"])
def test_one_workgroup_cycle(n, bc, precision):
    _check(n, bc, precision)


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("n", [(7, 9), (9, 11), (16, 16), (20, 36), (64, 64), (5, 4, 3 + 2), (8, 12, 8), (16, 16, 16),
                               (128, 96), (24, 16, 20)], ids=str)
@pytest.mark.parametrize("bc", [None, WALLS], ids=["periodic", "walls"])
def test_one_workgroup_cycle_density(n, bc, precision):
    _check(n, bc, precision, density=True)


# 2D levels that no tile divides: edge tiles past periodic and other sides,
# a second ragged level, the last too low for any tile but 32 x 8, one to four
# sweeps (four: no tiles)
RAGGED = [(88, 72), (72, 88), (240, 176), (24, 208), (44, 100), (212, 20)]


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("bc", [None, WALLS, OPEN], ids=["periodic", "walls", "open"])
@pytest.mark.parametrize("n", RAGGED, ids=str)
def test_ragged_tiles(n, bc, precision):
    _check(n, bc, precision)


@pytest.mark.parametrize("nu", [1, 3, 4])
@pytest.mark.parametrize("bc", [None, OPEN], ids=["periodic", "open"])
def test_ragged_tiles_sweeps(bc, nu):
    _check((88, 72), bc, nu=nu)


@pytest.mark.parametrize("precision", ["fp64", "mixed", "mixed-flexible"])
@pytest.mark.parametrize("bc", [None, WALLS], ids=["periodic", "walls"])
@pytest.mark.parametrize("n", [(88, 72), (72, 104), (24, 208)], ids=str)
def test_ragged_tiles_density(n, bc, precision):
    _check(n, bc, precision, density=True)


@pytest.mark.parametrize("precision", ["fp64", "mixed", "mixed-flexible"])
@pytest.mark.parametrize("n", [(96, 96), (88, 72), (24, 208)], ids=str)
def test_tiles_stretched(n, precision):
    _check(n, WALLS, precision, stretch=2.0)


# fused 3D levels: a small finest level, frames several periods wide, the
# fewest planes the march takes, chunks that do not divide the planes, and
# one plane pair too few (unfused)
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("nu", [1, 2])
@pytest.mark.parametrize("n", [(40, 24, 28), (8, 48, 16), (8, 8, 80), (12, 20, 24), (32, 40, 36), (32, 40, 8)], ids=str)
def test_fused_3d_levels(n, nu, precision):
    _check(n, None, precision, nu=nu)


# 3D CG update beyond the one-workgroup solve: periodic columns that do not
# divide the grid in x or y, and the form for other sides; the coarsest
# levels hold 540, 240 and 408 cells (dense inverse)
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("bc", [None, WALLS, OPEN], ids=["periodic", "walls", "open"])
@pytest.mark.parametrize("n", [(72, 20, 24), (24, 20, 32), (136, 12, 16)], ids=str)
def test_cg_update_3d(n, bc, precision):
    _check(n, bc, precision)


# the finest 2D level with just enough large tiles (418, 400) and just too
# few (384, 320), at the rtol of a run
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("bc", [None, WALLS], ids=["periodic", "walls"])
@pytest.mark.parametrize("n", [(704, 608), (640, 640), (768, 512), (640, 512)], ids=str)
def test_finest_tile_size(n, bc, precision):
    _check(n, bc, precision, rtol=1e-10)


# grids of several thousand finest tiles or cell blocks, which start while
# the first one ends the solve: the same solution to the last bit each time
@pytest.mark.parametrize("precision", ["fp64", "mixed-flexible"])
@pytest.mark.parametrize("n,bc", [((4096, 1024), None), ((2048, 2048), WALLS)], ids=["periodic", "walls"])
def test_large_solve_is_reproducible(n, bc, precision):
    import torch
    from paper_2603_01727_amd import Solver
    bc = None if bc is None else bc[:2]
    s = Solver(n, (1.0, n[1] / n[0]), bc=bc, Re=10.0, dt=1e-3, precision=precision, poisson_rtol=1e-10)
    b = torch.randn(n[1], n[0], dtype=torch.float64, device="cuda", generator=torch.Generator("cuda").manual_seed(9))
    print("reproducible", n, bc, precision, flush=True)
    first, info = s.project(b)
    first = first.clone()
    assert info["relres"] <= 1e-10
    for _ in range(6):
        again, info2 = s.project(b)
        assert info2 == info and torch.equal(again, first)
    s.close()


# 3D CG update with a density: columns of 72 = 64 + 8 cells, rows of 12 = 8 + 4
# and 28 = 3 * 8 + 4, faces of periodic and other sides, coarsest levels of
# at most 128 cells
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("bc", [None, WALLS, OPEN], ids=["periodic", "walls", "open"])
@pytest.mark.parametrize("n", [(72, 24, 16), (24, 12, 28), (12, 28, 24)], ids=str)
def test_cg_update_3d_density(n, bc, precision):
    _check(n, bc, precision, density=True)


# tolerances from none at all (the zero start passes) to one that only the
# iteration limit ends: the count of iterations queued before the outcome is
# read stays a number
@pytest.mark.parametrize("rtol,iters", [(math.inf, 0), (2.0, 0), (1e-320, None)], ids=str)
@pytest.mark.parametrize("n", [(96, 80), (24, 20, 32)], ids=str)
def test_extreme_tolerances(n, rtol, iters):
    from paper_2603_01727_amd import LowMachError, Solver, lib
    s = Solver(n, (1.0,) * len(n), Re=10.0, dt=1e-3, poisson_rtol=1e-10, poisson_maxit=12)
    b = np.random.default_rng(5).standard_normal(tuple(reversed(n)))
    print("tolerance", n, rtol, flush=True)
    if iters is None:
        with pytest.raises(LowMachError) as e:
            s.project(b, rtol=rtol)
        assert e.value.status == lib.LM_ENOCONV
    else:
        P, info = s.project(b, rtol=rtol)
        assert info["iters"] == iters and not P.any()
    s.close()


# the timing hook on grids that store A p (flexible CG) and that do not: every
# class still runs, on vectors of its own, and the next solve is unharmed
@pytest.mark.parametrize("precision", ["fp64", "mixed", "mixed-flexible"])
@pytest.mark.parametrize("n", [(96, 80), (24, 20, 32)], ids=str)
def test_kernel_timing_hook(n, precision):
    import ctypes as C
    import torch
    from paper_2603_01727_amd import Solver
    s = Solver(n, (1.0,) * len(n), Re=10.0, dt=1e-3, precision=precision)
    one = torch.ones(tuple(reversed(n)), dtype=torch.float64, device="cuda")
    s.set(T=one, v=[one * 0.0] * len(n))
    b = torch.randn(one.shape, dtype=torch.float64, device="cuda", generator=torch.Generator("cuda").manual_seed(4))
    before, _ = s.project(b)
    before = before.clone()
    for which in range(8):
        print("hook", n, precision, which, flush=True)
        ms = C.c_double(-1.0)
        assert s.lib.lm_bench_kernel(s.ctx, which, 2, C.byref(ms)) == 0
        assert ms.value > 0.0
    after, _ = s.project(b)
    assert torch.equal(before, after)
    s.close()

"""Multigrid level kernels at the sizes where they can go wrong, through the
pressure solve (lm_project) against the oracle's exact solve.

Tolerance: the solve stops at relative residual rtol, so the relative error
is at most kappa rtol, kappa = lambda_max / lambda_min of the operator (times
the density ratio), plus the same bound for rounding at 1e-15."""
import math

import numpy as np
import pytest

from oracle import Grid, PoissonSolver, beta_inv_rho
from workloads import variable_coefficient_problem
from _cases import rel_l2

pytestmark = pytest.mark.gpu
RTOL = 1e-13
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


def _check(n, bc=None, precision="fp64", density=False):
    from paper_2603_01727_amd import Solver
    L = tuple(1.0 + 0.25 * d for d in range(len(n)))
    bc = None if bc is None else bc[:len(n)]
    rho, b = variable_coefficient_problem(n, L, seed=3 + sum(n), kmax=2, m=6)
    g = Grid(n, L, bc=None if bc is None else tuple(bc))
    print("levels", n, bc, precision, "density" if density else "", flush=True)
    want = PoissonSolver(g, beta_inv_rho(g, rho) if density else None).solve(b)[0]
    s = Solver(n, L, bc=bc, Re=10.0, dt=1e-3, precision=precision, poisson_rtol=RTOL, poisson_maxit=400,
               variable_coefficient=density)
    got, info = s.project(b, rho=rho if density else None)
    s.close()
    err, tol = rel_l2(got, want), _kappa(n, L, bc) * (4.0 if density else 1.0) * (RTOL + 1e-15)
    print(err, tol, info, flush=True)
    assert info["relres"] <= RTOL
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

"""Iteration counts of the pressure solve against the same method in numpy.

CG repairs most errors of a smoother, a restriction or a halo: the solution
still converges, in more iterations. The reference below is the method
itself (red-black sweeps, averages of the children, piecewise constant
corrections, dense coarsest inverse, preconditioned CG from zero) on whole
arrays in FP64, so that in exact arithmetic the counts are equal. Rounding
(FP32 in the mixed cycles) can move the residual across the tolerance by
one iteration at most where it falls by a factor of two or more in each:
the counts may differ by 1."""
import math

import numpy as np
import pytest

from oracle import Grid, PoissonSolver, beta_inv_rho
from workloads import tanh_stretched_faces, variable_coefficient_problem
from _cases import rel_l2

pytestmark = pytest.mark.gpu
WALLS = [("noslip", "noslip"), ("slip", "slip"), ("noslip", "slip")]
OPEN = [("slip", "slip"), ("inflow", "outflow"), ("periodic", "periodic")]
RTOL = 1e-9


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


class _Level:
    """L = -A on one level: coefficients of every cell's low face, x first."""

    def __init__(self, low):
        self.low = low
        nd = len(low)
        self.ax = [nd - 1 - d for d in range(nd)]
        self.high = [np.roll(c, -1, self.ax[d]) for d, c in enumerate(low)]
        self.diag = sum(low) + sum(self.high)
        self.red = sum(np.indices(low[0].shape)) % 2 == 0

    def nbs(self, x):
        return sum(self.low[d] * np.roll(x, 1, self.ax[d]) + self.high[d] * np.roll(x, -1, self.ax[d])
                   for d in range(len(self.ax)))

    def apply(self, x):
        return self.diag * x - self.nbs(x)

    def sweep(self, x, b, colour):
        return np.where(self.red == colour, (b + self.nbs(x)) / self.diag, x)


def _children(a):
    """Mean of the 2^d children of every coarse cell."""
    for ax in range(a.ndim):
        a = a.reshape(a.shape[:ax] + (a.shape[ax] // 2, 2) + a.shape[ax + 1:]).mean(ax + 1)
    return a


def _parents(a):
    for ax in range(a.ndim):
        a = np.repeat(a, 2, ax)
    return a


def _hierarchy(n, L, bc, rho, faces):
    nd, levels, l = len(n), [], 0
    w = None if faces is None else [np.diff(f) for f in faces]
    while True:
        shape = tuple(reversed(n))
        low = []
        for d in range(nd):
            ax = nd - 1 - d
            if w is not None:  # volume-weighted: face length / distance of the centres, a quarter per level
                dist = 0.5 * (w[d] + np.roll(w[d], 1))
                other = w[1 - d].reshape((-1, 1) if d == 0 else (1, -1))
                c = other / dist.reshape((1, -1) if d == 0 else (-1, 1)) * 0.25 ** l
            else:
                c = np.full(shape, (n[d] / L[d]) ** 2)
                if rho is not None:
                    c = c * 2.0 / (rho + np.roll(rho, 1, ax))
            c = np.array(np.broadcast_to(c, shape))
            if bc is not None and bc[d][0] != "periodic":
                c[tuple(slice(0, 1) if a == ax else slice(None) for a in range(nd))] = 0.0
            low.append(c)
        levels.append(_Level(low))
        if any(q % 2 or q // 2 < 2 for q in n) or np.prod(n) <= 64:
            break
        n = tuple(q // 2 for q in n)
        rho = None if rho is None else _children(rho)
        w = None if w is None else [q[::2] + q[1::2] for q in w]
        l += 1
    A = np.array([levels[-1].apply(e.reshape(shape)).ravel() for e in np.eye(int(np.prod(n)))])
    return levels, np.linalg.pinv(0.5 * (A + A.T), rcond=1e-12, hermitian=True)


def _cycle(levels, pinv, nu, b, l=0):
    if l == len(levels) - 1:
        return (pinv @ b.ravel()).reshape(b.shape)
    A, x = levels[l], np.zeros_like(b)
    for _ in range(nu):
        x = A.sweep(A.sweep(x, b, True), b, False)
    x = x + _parents(_cycle(levels, pinv, nu, _children(b - A.apply(x)), l + 1))
    for _ in range(nu):
        x = A.sweep(A.sweep(x, b, False), b, True)
    return x


def _count(n, L, bc, rho, faces, b, nu):
    levels, pinv = _hierarchy(n, L, bc, rho, faces)
    if faces is None:
        c = -(b - b.mean())
    else:
        v = np.outer(np.diff(faces[1]), np.diff(faces[0]))
        c = -(b - (b * v).sum() / v.sum()) * v
    r, cc = c.copy(), (c * c).sum()
    p, g_old, k = 0.0, 1.0, 0
    while (r * r).sum() > RTOL ** 2 * cc:
        z = _cycle(levels, pinv, nu, r)
        g = (r * z).sum()
        p = z + (g / g_old if k else 0.0) * p
        q = levels[0].apply(p)
        r = r - g / (p * q).sum() * q
        g_old, k = g, k + 1
        assert k < 200
    return k


def _check(n, bc=None, nu=2, precision="fp64", density=False, stretch=0.0, apart=1):
    from paper_2603_01727_amd import Solver
    L = tuple(q / max(n) for q in n)  # cells of equal sides: few iterations
    bc = None if bc is None else bc[:len(n)]
    rho = variable_coefficient_problem(n, L, seed=3 + sum(n), kmax=2, m=6)[0] if density else None
    faces = [tanh_stretched_faces(q, stretch, l) for q, l in zip(n, L)] if stretch else None
    b = np.random.default_rng(sum(n)).standard_normal(tuple(reversed(n)))
    print("iterations", n, bc, nu, precision, density, stretch, flush=True)
    want = _count(n, L, bc, rho, faces, b, nu)
    s = Solver(n, L, bc=bc, Re=10.0, dt=1e-3, precision=precision, poisson_rtol=RTOL, mg_nu=nu,
               variable_coefficient=density, faces=faces)
    got, info = s.project(b, rho=rho)
    s.close()
    print(want, info, flush=True)
    assert abs(info["iters"] - want) <= apart
    g = Grid(n, L, bc=None if bc is None else tuple(bc), faces=faces)
    exact = PoissonSolver(g, beta_inv_rho(g, rho) if density else None).solve(b)[0]
    # relative error <= condition of L times the tolerance; 4 nd (max n)^2 / 4 and the ratios of density and widths
    assert rel_l2(got, exact) <= len(n) * max(n) ** 2 * (4.0 if density else 1.0) * max(stretch, 1.0) ** 4 * RTOL


PRECISIONS = ["fp64", "mixed", "mixed-flexible"]

# one workgroup; whole tiles; edge tiles, the last too low for any but 32 x 8;
# too narrow for any tile; fused 3D levels, frames of several periods; 3D
# with sides
ONE = [((64, 64), None), ((30, 22), WALLS), ((16, 16, 16), None), ((20, 12, 14), OPEN),
       ((128, 96), None), ((768, 512), WALLS), ((704, 608), None),
       ((88, 72), None), ((240, 176), WALLS), ((212, 20), OPEN),
       ((20, 212), None), ((20, 212), OPEN),
       ((40, 24, 28), None), ((8, 48, 16), None), ((64, 64, 32), None),
       ((24, 20, 32), WALLS), ((72, 20, 24), OPEN)]


@pytest.mark.parametrize("precision", PRECISIONS)
@pytest.mark.parametrize("n,bc", ONE, ids=str)
def test_iterations(n, bc, precision):
    _check(n, bc, precision=precision)


# the forms without tiles (four sweeps; sides too narrow) and the others, with
# a density and on stretched grids
@pytest.mark.parametrize("precision", PRECISIONS)
@pytest.mark.parametrize("n,bc,nu", [((64, 48), WALLS, 2), ((88, 72), OPEN, 2), ((88, 72), None, 4), ((88, 72), OPEN, 4),
                                     ((16, 264), WALLS, 2), ((24, 16, 20), None, 2), ((24, 12, 28), OPEN, 2)], ids=str)
def test_iterations_density(n, bc, nu, precision):
    _check(n, bc, nu, precision, density=True)


@pytest.mark.parametrize("precision", PRECISIONS)
@pytest.mark.parametrize("n,nu", [((48, 48), 2), ((96, 96), 2), ((88, 72), 4), ((16, 264), 2)], ids=str)
def test_iterations_stretched(n, nu, precision):
    _check(n, WALLS, nu, precision, stretch=1.5)


@pytest.mark.parametrize("precision", PRECISIONS)
@pytest.mark.parametrize("n,bc,nu", [((88, 72), OPEN, 1), ((88, 72), None, 3), ((88, 72), WALLS, 4), ((40, 24, 28), None, 1),
                                     ((24, 20, 32), None, 3)], ids=str)
def test_iterations_sweeps(n, bc, nu, precision):
    _check(n, bc, nu, precision)


# the dense inverse of a grid that is its own coarsest level, its columns in
# runs of 9, 32, 88 = 2 * 32 + 24, 315, 729 (two passes of rows), 513 and 1023.
# Exact: one iteration; rounded to FP32 each leaves a residual of about
# 2^-24 times the condition of L
@pytest.mark.parametrize("precision", PRECISIONS)
@pytest.mark.parametrize("n", [(5, 13), (5, 5, 5), (5, 5, 7), (9, 7, 5), (9, 9, 9), (9, 57), (31, 33)], ids=str)
def test_iterations_dense(n, precision):
    left = 2.0 ** (-53 if precision == "fp64" else -24) * len(n) * max(n) ** 2
    _check(n, WALLS, precision=precision, apart=max(1, math.ceil(math.log(RTOL) / math.log(left)) - 1))

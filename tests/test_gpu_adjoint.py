"""GPU checks of checkpoint/restart and of the hand-written adjoint.

* save/load of the state reproduces a run bit for bit;
* dot-product test of one adjoint step against the oracle's complex-step
  tangent of the same step: <ybar, J dx> = <J^T ybar, dx> for random
  cotangents ybar of every output and random directions dx of every input,
  in 2D and 3D (also with buoyancy and Sutherland's conductivity);
* gradient of the final kinetic energy with respect to T0 (autograd
  Function, checkpointed) against the oracle's complex-step derivative and
  against central finite differences of the GPU forward (h = 1e-6, 16
  seeded directions, <= 1e-6 relative).
Every Poisson solve is converged to 1e-14 so that solver error stays below
the finite-difference resolution; dt is fixed.
"""
import math
import time

import numpy as np
import pytest

from oracle import Grid, Oracle, Params
from oracle import tangent as tg
from workloads.ics import c1_case, c3_case, c5_case, fd_directions

pytestmark = pytest.mark.gpu
RTOL = 1e-14


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _dt(case):
    nd = case.ndim
    g = Grid(case.n[:nd], case.L[:nd], bc=case.bc, bnd=case.bnd)
    o = Oracle(g, Params(Re=case.params["Re"], Pr=case.params["Pr"], cfl=case.params["cfl"], **_flame(case)))
    o.initial_state(case.T, case.v, Z=case.Z, H=case.H)
    return o.dt


def _flame(case):
    """The reacting-flow parameters of a case (empty without reaction)."""
    keys = ("reacting", "S", "qs", "eps", "tol", "Le_F", "Le_O")
    return {k: case.params[k] for k in keys if k in case.params}


def _solver(case, dt, with_adjoint=True, rtol=RTOL, sutherland_C=0.0, inv_Fr2=0.0):
    from paper_2603_01727_amd import Solver
    nd = case.ndim
    return Solver(case.n[:nd], case.L[:nd], bc=case.bc, Re=case.params["Re"], Pr=case.params["Pr"], dt=dt,
                  poisson_rtol=rtol, poisson_maxit=400, with_adjoint=with_adjoint, sutherland_C=sutherland_C,
                  inv_Fr2=inv_Fr2, with_ib=case.ib is not None, Da_ib=case.params.get("Da_ib", 1.0),
                  **_flame(case))


def test_state_restart_is_bit_exact():
    import torch
    case = c1_case()
    print("restart c1", flush=True)
    s = _solver(case, 0.02, with_adjoint=False, rtol=1e-12)
    s.set(T=case.T, v=case.v)
    s.step(3)
    buf = s.save_state()
    s.step(4)
    a = s.get(device=False)
    s.load_state(buf)
    s.step(4)
    b = s.get(device=False)
    s2 = _solver(case, 0.02, with_adjoint=False, rtol=1e-12)
    s2.set(T=case.T + 1.0, v=case.v)          # a different state, overwritten
    s2.load_state(buf.clone())
    s2.step(4)
    c = s2.get(device=False)
    for k in ("rho", "H", "T", "P"):
        assert np.array_equal(a[k], b[k]) and np.array_equal(a[k], c[k]), k
    for d in range(2):
        assert np.array_equal(a["v"][d], b["v"][d]) and np.array_equal(a["v"][d], c["v"][d])
        assert np.array_equal(a["F"][d], c["F"][d])
    assert s2.state_size() == buf.numel()
    torch.cuda.synchronize()


def _faces(f, ax):
    return np.concatenate([np.take(f, [-1], axis=ax), f], axis=ax)


def _dot(a, b):
    out = 0.0
    for k in a:
        if k not in b:
            continue
        x, y = a[k], b[k]
        if isinstance(x, list):
            out += sum(float(np.sum(np.asarray(p) * np.asarray(q))) for p, q in zip(x, y))
        else:
            out += float(np.sum(np.asarray(x) * np.asarray(y)))
    return out


def _clear_fixed_faces(g, case, F, direction=False):
    """Face arrays restricted to their free entries. Face 0 of a periodic
    direction duplicates face n: a cotangent carries nothing there (the
    library holds the pair's cotangent at face n), and a direction of the
    state (``direction``) moves both alike, as every state the step makes
    has them equal. Wall faces carry a constant flux: zero in both."""
    for d in range(case.ndim):
        lo = [slice(None)] * case.ndim
        hi = [slice(None)] * case.ndim
        lo[g.axis(d)] = 0
        hi[g.axis(d)] = -1
        if case.bc[d][0] == "periodic":
            F[d][tuple(lo)] = F[d][tuple(hi)] if direction else 0.0
        else:
            F[d][tuple(lo)] = 0.0
            if case.bc[d][1] != "outflow":      # an outflow face flux is free
                F[d][tuple(hi)] = 0.0


def _dot_product_check(case, history, suth=0.0, inv_Fr2=0.0, seed=100):
    """One step back on the GPU against the complex-step tangent of the same
    step in the oracle, per input component."""
    nd = case.ndim
    dt = 0.5 * _dt(case)
    g = Grid(case.n[:nd], case.L[:nd], bc=case.bc, bnd=case.bnd)
    p = Params(Re=case.params["Re"], Pr=case.params["Pr"], dt=dt, sutherland_C=suth, inv_Fr2=inv_Fr2,
               Da_ib=case.params.get("Da_ib", 1.0), **_flame(case))
    react = p.reacting
    o = Oracle(g, p, ib=case.ib)
    st = o.initial_state(case.T, case.v, Z=case.Z, H=case.H)
    nhist = 1 if history else 0
    st = tg.with_eos(o, o.run(st, nhist))
    s = _solver(case, dt, sutherland_C=suth, inv_Fr2=inv_Fr2)
    for (d, side), data in (case.bnd or {}).items():
        s.set_side(d, side, v=data.get("v"), Z=data.get("Z"), H=data.get("H"), F=data.get("F"),
                   wall=data.get("wall"))
    s.set(T=case.T, H=case.H if case.T is None else None, v=case.v, Z=case.Z, ib=case.ib)
    if nhist:
        s.step(nhist)
    rng = np.random.default_rng(seed)
    # cotangents of the step's outputs (face 0 of a periodic face array is a
    # duplicate of face n and carries none; wall faces carry a constant flux)
    ybar = {"H": rng.normal(size=g.shape), "v": [rng.normal(size=g.shape) for _ in range(nd)],
            "rho_prev": rng.normal(size=g.shape), "R_H": rng.normal(size=g.shape),
            "R_v": [rng.normal(size=g.shape) for _ in range(nd)]}
    ybar["F"] = [_faces(rng.normal(size=g.shape), g.axis(d)) for d in range(nd)]
    if react:
        ybar["Z"] = rng.normal(size=g.shape)
        ybar["R_Z"] = rng.normal(size=g.shape)
    _clear_fixed_faces(g, case, ybar["F"])
    s.adjoint_set(**ybar)
    t0 = time.time()
    s.step_adjoint()
    xbar = s.adjoint_get(device=False)
    print("step_adjoint", time.time() - t0, flush=True)
    comps = ["H", "v", "F"] + (["rho_prev", "R_H", "R_v"] if history else [])
    if react:
        comps += ["Z"] + (["R_Z"] if history else [])
    for k in comps:
        if k == "F":
            dx = {k: [_faces(rng.normal(size=g.shape), g.axis(d)) for d in range(nd)]}
            _clear_fixed_faces(g, case, dx[k], direction=True)
        elif k in ("v", "R_v"):
            dx = {k: [rng.normal(size=g.shape) for _ in range(nd)]}
        elif k == "Z":
            dx = {k: 0.1 * rng.normal(size=g.shape)}
        else:
            dx = {k: rng.normal(size=g.shape)}
        ydot = tg.step_tangent(o, st, dx)
        lhs = _dot(ybar, ydot)
        rhs = _dot(xbar, dx)
        print(k, lhs, rhs, abs(lhs - rhs) / abs(lhs), flush=True)
        assert abs(lhs - rhs) <= 1e-9 * abs(lhs), (k, lhs, rhs)


@pytest.mark.parametrize("shape,history,suth,fr", [((72, 80), False, 0.0, 0.0), ((72, 80), True, 0.0, 0.0),
                                                   ((64, 64), True, 0.0, 0.0),
                                                   ((64, 64), True, 110.5 / 600.0, 0.0),
                                                   ((64, 64), True, 0.0, 0.5)],
                         ids=["72x80", "72x80-hist", "64-hist", "64-hist-sutherland", "64-hist-buoyancy"])
def test_adjoint_step_dot_product_against_oracle_tangent(shape, history, suth, fr):
    """2D: also with Sutherland's conductivity (Eq 4.12) and with buoyancy
    (1/Fr^2 = 0.5, Eq 2.43)."""
    ny, nx = shape
    case = c5_case(n=nx)
    if ny != nx:
        from workloads.ics import fourier_temperature, solenoidal_velocity
        L = (2 * math.pi, 2 * math.pi)
        rng = np.random.default_rng(5)
        case.T = fourier_temperature((nx, ny), L, rng, 8, 3.0)
        case.v = solenoidal_velocity((nx, ny), L, rng, 8, 0.1)
        case.n = (nx, ny, 1)
    print("adjoint dot", shape, history, suth, fr, flush=True)
    _dot_product_check(case, history, suth, fr, seed=100 + nx + ny)


def _case3d(n, seed=8, amp=3.0):
    """Periodic 2*pi box in 3D with n = (nx, ny, nz): T = 1 + amp fhat
    (24 modes, |k| <= 3), solenoidal velocity rms 0.1, Re = 300."""
    from workloads.ics import Case, fourier_temperature, solenoidal_velocity
    L = (2 * math.pi,) * 3
    rng = np.random.default_rng(seed)
    T = fourier_temperature(n, L, rng, 3, amp, m=24)
    v = solenoidal_velocity(n, L, rng, 3, 0.1, m=24)
    return Case("adjoint_3d", 3, tuple(n), L, (("periodic", "periodic"),) * 3,
                dict(Re=300.0, Pr=0.7, cfl=0.3), T, v, nsteps=1)


@pytest.mark.parametrize("n,history,suth,fr", [((12, 10, 8), False, 0.0, 0.0), ((12, 10, 8), True, 0.0, 0.5),
                                               ((20, 18, 16), True, 110.5 / 600.0, 0.0),
                                               ((24, 16, 20), True, 0.0, 0.5)],
                         ids=["12x10x8", "12x10x8-hist-buoyancy", "20x18x16-hist-sutherland",
                              "24x16x20-hist-buoyancy"])
def test_adjoint_step_dot_product_3d(n, history, suth, fr):
    """3D: the 3^3-cell residual gather, the three-component projection and
    Adams transposes; 960 cells take the one-workgroup pressure solve,
    the larger grids the multi-kernel one."""
    print("adjoint dot 3d", n, history, suth, fr, flush=True)
    _dot_product_check(_case3d(n), history, suth, fr, seed=200 + sum(n))


def _with_body(case, seed, Da=0.05, source=False):
    """The case with a penalised body (Eq 3.30-3.32): a ball of radius 1.2
    at the box centre turning rigidly about z with unit angular speed
    (v_ib = (-y, x, 0) about the centre, zero beyond the ball), H_ib = 2.5
    (and Z_ib = 0.5 in reacting flow); with ``source`` also a seeded mass source S_m ~ 0.1 N(0, 1)."""
    nd = case.ndim
    from workloads.ics import cell_centres
    xs = cell_centres(case.n[:nd], case.L[:nd])
    xs = [x - 0.5 * Lq for x, Lq in zip(xs, case.L[:nd])]
    X = np.broadcast_arrays(*xs)
    r2 = sum(x * x for x in X)
    chi = (r2 < 1.2 ** 2).astype(np.uint8)
    vib = [np.where(chi == 1, -X[1], 0.0), np.where(chi == 1, X[0], 0.0)] + ([np.zeros(chi.shape)] if nd == 3 else [])
    ib = dict(chi=chi, v_ib=vib, H_ib=np.full(chi.shape, 2.5))
    if case.Z is not None:
        ib["Z_ib"] = np.full(chi.shape, 0.5)
    if source:
        ib["Sm"] = 0.1 * np.random.default_rng(seed).normal(size=chi.shape)
    case.ib = ib
    case.params = dict(case.params, Da_ib=Da)
    return case


@pytest.mark.parametrize("dim,history,source", [(2, True, False), (2, False, True), (3, True, True)],
                         ids=["2d-64-hist", "2d-64-source", "3d-16x14x12-hist-source"])
def test_adjoint_step_dot_product_immersed_body(dim, history, source):
    """With a penalised body: the body terms of R_H and R_v enter the
    residual gather (mask and targets are constants); S_m has no
    cotangent."""
    case = c5_case(n=64) if dim == 2 else _case3d((16, 14, 12), seed=11)
    case = _with_body(case, seed=31, source=source)
    print("adjoint dot body", dim, history, source, flush=True)
    _dot_product_check(case, history, seed=300 + dim)


def test_ke_gradient_immersed_body_against_oracle_complex_step():
    """2D 64^2 with the turning body, 6 steps, checkpoints every 2: J and its
    T0-gradient along 3 seeded directions against the oracle's complex
    step."""
    import torch
    from paper_2603_01727_amd.adjoint import final_kinetic_energy
    nsteps, k = 6, 2
    case = _with_body(c5_case(n=64), seed=32, source=True)
    dt = _dt(case)
    print("ke gradient with body", nsteps, flush=True)
    s = _solver(case, dt)
    T0 = torch.tensor(case.T, dtype=torch.float64, device="cuda", requires_grad=True)
    v0 = [torch.tensor(a, dtype=torch.float64, device="cuda") for a in case.v]
    J = final_kinetic_energy(s, T0, v0, nsteps, k, ib=case.ib)
    J.backward()
    grad = T0.grad.cpu().numpy()
    g = Grid(case.n[:2], case.L[:2], bc=case.bc)
    p = Params(Re=case.params["Re"], Pr=case.params["Pr"], dt=dt, Da_ib=case.params["Da_ib"])
    Jo = tg.final_kinetic_energy(g, p, case.T, case.v, nsteps, ib=case.ib)
    print("J", J.item(), Jo, flush=True)
    assert abs(J.item() - Jo) <= 1e-12 * abs(Jo)
    for d in fd_directions(case.T.shape, k=3):
        cs = tg.ke_directional(g, p, case.T, case.v, d, nsteps, ib=case.ib)
        ad = float(np.sum(grad * d))
        print(cs, ad, abs(ad - cs) / abs(cs), flush=True)
        assert abs(ad - cs) <= 1e-9 * abs(cs)


@pytest.mark.parametrize("n,history,body", [((64, 64), False, False), ((64, 64), True, False),
                                             ((72, 56), True, True), ((12, 10, 8), True, False),
                                             ((16, 14, 12), True, True)],
                         ids=["2d-64", "2d-64-hist", "2d-72x56-hist-body", "3d-12x10x8-hist",
                              "3d-16x14x12-hist-body"])
def test_adjoint_step_dot_product_reacting(n, history, body):
    """Reacting mixture (Z spans the flame level Z = 1, Le_F = 0.8,
    Le_O = 1.2): the dual gather carries Z (the flame map T(Z, H) of
    Eq 3.42, theta_eps and the Lewis factors of Eq 3.34-3.35, the Z
    transport and its body term), the tail the Z Adams updates and
    d rho/dZ; per input component including Z and R_Z."""
    from workloads.ics import reacting_periodic_case
    case = reacting_periodic_case(n, seed=13)
    if body:
        case = _with_body(case, seed=33, source=True)
    print("adjoint dot reacting", n, history, body, flush=True)
    _dot_product_check(case, history, seed=400 + sum(n))


def test_ke_gradient_reacting_against_oracle_complex_step():
    """Reacting 2D 64^2, 6 steps, checkpoints every 2: J, its T0-gradient
    (Z0 fixed) and the Z0-gradient from the initial-state transpose
    (H0 = T0/qs - F~(Z0)) along seeded directions against the oracle's
    complex step."""
    import torch
    from paper_2603_01727_amd.adjoint import Trajectory
    from workloads.ics import reacting_periodic_case
    nsteps, k = 6, 2
    case = reacting_periodic_case((64, 64), seed=14)
    dt = _dt(case)
    print("ke gradient reacting", nsteps, flush=True)
    s = _solver(case, dt)
    traj = Trajectory(s, nsteps, k)
    dev = lambda a: torch.tensor(a, dtype=torch.float64, device="cuda")
    J = traj.forward(dev(case.T), [dev(a) for a in case.v], dev(case.Z))
    Tb, vb, Zb = traj.backward()
    Tb, Zb = Tb.cpu().numpy(), Zb.cpu().numpy()
    g = Grid(case.n[:2], case.L[:2], bc=case.bc)
    p = Params(Re=case.params["Re"], Pr=case.params["Pr"], dt=dt, **_flame(case))
    Jo = tg.final_kinetic_energy(g, p, case.T, case.v, nsteps, Z0=case.Z)
    print("J", J, Jo, flush=True)
    assert abs(J - Jo) <= 1e-12 * abs(Jo)
    zero = np.zeros(case.T.shape)
    for q, d in enumerate(fd_directions(case.T.shape, k=4)):
        if q % 2 == 0:
            cs = tg.ke_directional(g, p, case.T, case.v, d, nsteps, Z0=case.Z)
            ad = float(np.sum(Tb * d))
        else:
            d = 0.1 * d
            cs = tg.ke_directional(g, p, case.T, case.v, zero, nsteps, Z0=case.Z, dZ=d)
            ad = float(np.sum(Zb * d))
        print("T0" if q % 2 == 0 else "Z0", cs, ad, abs(ad - cs) / abs(cs), flush=True)
        assert abs(ad - cs) <= 1e-9 * abs(cs)


def _walls_case(kind, seed=21):
    """Boxes with wall sides (section 3.6, Eq 3.43), random T in [1, 3] and
    velocity rms 0.1 (the fields need not meet the wall conditions: the
    step's ghosts and wall fluxes impose them):
    'channel'  2D 64 x 48, periodic in x, slip walls in y;
    'cavity'   2D 48 x 40 unit box, no-slip walls, the x walls isothermal
               (T = 1.4 and 0.6: H = T + 1), adiabatic y walls;
    'duct3d'   3D 16 x 14 x 12, periodic in x, slip walls in y, no-slip in z;
    'box3d'    3D 12 x 10 x 8, no-slip walls on every side."""
    from workloads.ics import Case, fourier_temperature, solenoidal_velocity
    shapes = {"channel": ((64, 48), (2 * math.pi, 1.5 * math.pi), ("periodic", "slip")),
              "cavity": ((48, 40), (1.0, 1.0), ("noslip", "noslip")),
              "duct3d": ((16, 14, 12), (2 * math.pi,) * 3, ("periodic", "slip", "noslip")),
              "box3d": ((12, 10, 8), (2 * math.pi,) * 3, ("noslip", "noslip", "noslip"))}
    n, L, kinds = shapes[kind]
    rng = np.random.default_rng(seed)
    T = fourier_temperature(n, L, rng, 3, 2.0, m=24)
    v = solenoidal_velocity(n, L, rng, 3, 0.1, m=24)
    bc = tuple((k, k) for k in kinds)
    bnd = None
    if kind == "cavity":
        bnd = {(0, 0): dict(H=np.full(n[1], 2.4)), (0, 1): dict(H=np.full(n[1], 1.6))}
    return Case(f"walls_{kind}", len(n), tuple(n) + (1,) * (3 - len(n)), L + (1.0,) * (3 - len(n)), bc,
                dict(Re=200.0, Pr=0.7, cfl=0.3), T, v, bnd=bnd, nsteps=1)


@pytest.mark.parametrize("kind,history,fr,react", [("channel", False, 0.0, False), ("channel", True, 0.5, False),
                                                   ("cavity", True, 0.5, False), ("channel", True, 0.0, True),
                                                   ("duct3d", True, 0.5, False), ("box3d", True, 0.0, True)],
                         ids=["channel", "channel-hist-buoyancy", "cavity-hist-buoyancy", "channel-hist-reacting",
                              "duct3d-hist-buoyancy", "box3d-hist-reacting"])
def test_adjoint_step_dot_product_walls(kind, history, fr, react):
    """Slip and no-slip walls, isothermal or adiabatic: the residual gather
    reads ghosts by the forward's rules (mirrors of interior cells, the
    wall conductivity 2 kappa(T_w) - kappa(T) at isothermal walls), wall
    faces carry a constant flux, the projection transpose takes the
    extrapolated pressure ghost and the right-hand side the one-sided face
    sums at walls."""
    case = _walls_case(kind)
    if react:
        from workloads.ics import reacting_periodic_case
        r = reacting_periodic_case(case.n[:case.ndim], seed=22)
        case.Z = r.Z
        case.params = dict(r.params, Re=case.params["Re"], cfl=case.params["cfl"])
    print("adjoint dot walls", kind, history, fr, react, flush=True)
    _dot_product_check(case, history, inv_Fr2=fr, seed=500 + len(kind))


def _open_case(kind, seed=41):
    """Open boxes (inflow at the low end of the last direction, outflow at
    its high end), random T in [1, 3], velocity rms 0.1 plus a mean stream
    of 0.5 along that direction:
    'channel'  2D 48 x 64, periodic in x;
    'duct3d'   3D 12 x 10 x 16, slip walls in x, periodic in y.
    The inflow carries v = 0.5 along the stream, T = 1.5 (H = 2.5) and the
    matching mass flux rho v = (p0/T) 0.5."""
    from workloads.ics import Case, fourier_temperature, solenoidal_velocity
    n, L, kinds = {"channel": ((48, 64), (2 * math.pi, 2.5 * math.pi), ("periodic",)),
                   "duct3d": ((12, 10, 16), (2 * math.pi,) * 3, ("slip", "periodic"))}[kind]
    nd = len(n)
    rng = np.random.default_rng(seed)
    T = fourier_temperature(n, L, rng, 3, 2.0, m=24)
    v = solenoidal_velocity(n, L, rng, 3, 0.1, m=24)
    v[-1] = v[-1] + 0.5
    bc = tuple((k, k) for k in kinds) + (("inflow", "outflow"),)
    side = tuple(reversed(n[:-1]))
    vin = [np.zeros(side) for _ in range(nd)]
    vin[-1] = np.full(side, 0.5)
    bnd = {(nd - 1, 0): dict(v=vin, H=np.full(side, 2.5), F=np.full(side, 0.5 / 1.5))}
    return Case(f"open_{kind}", nd, tuple(n) + (1,) * (3 - nd), L + (1.0,) * (3 - nd), bc,
                dict(Re=200.0, Pr=0.7, cfl=0.3), T, v, bnd=bnd, nsteps=1)


@pytest.mark.parametrize("kind,history", [("channel", False), ("channel", True), ("duct3d", True),
                                          ("slot", False), ("slot", True)],
                         ids=["channel", "channel-hist", "duct3d-hist", "slot-flame", "slot-flame-hist"])
def test_adjoint_step_dot_product_open(kind, history):
    """Inflow and outflow sides (section 3.6): extrapolated outflow ghosts
    (Eq 3.43), the outflow face flux extrapolated from the momentum, and the
    transpose of the uniform outflow closure (sum(b) over the outflow area,
    section 3.3) after each adjoint solve. 'slot': the slot flame reduced to
    48 x 64 (burner walls and injector as a penalised body with a mass
    source, fuel Z = S + 1, footprint walls on the inflow side, slip side
    walls)."""
    if kind == "slot":
        case = c3_case(nx=48, ny=64, W=8, wall=2, wall_h=12, inj=2)
        # The slot flame holds Z = 0 and Z = S + 1 exactly in many cells, so
        # their mirrored inflow ghosts sit exactly on the ends of the ghost
        # clamp [0, S+1], where the step is not differentiable (the complex
        # clip of the oracle picks a side by the sign of the perturbation).
        # Keep the cells 1e-3 inside the range: the ghosts then lie strictly
        # outside it and are clamped on both sides alike.
        zmax = case.params["S"] + 1.0
        case.Z = np.clip(case.Z, 1e-3, zmax - 1e-3)
    else:
        case = _open_case(kind)
    print("adjoint dot open", kind, history, flush=True)
    _dot_product_check(case, history, seed=600 + len(kind))


def test_ke_gradient_open_channel_against_oracle_complex_step():
    """The open channel (inflow / outflow), 6 steps with checkpoints every 2:
    J and its T0-gradient along 3 seeded directions against the oracle's
    complex step (the initial-state transpose takes the extrapolated
    outflow face flux; the closure enters every step)."""
    import torch
    from paper_2603_01727_amd.adjoint import final_kinetic_energy
    nsteps, k = 6, 2
    case = _open_case("channel", seed=42)
    dt = _dt(case)
    print("ke gradient open channel", nsteps, flush=True)
    s = _solver(case, dt)
    for (d, side), data in case.bnd.items():
        s.set_side(d, side, v=data.get("v"), H=data.get("H"), F=data.get("F"))
    T0 = torch.tensor(case.T, dtype=torch.float64, device="cuda", requires_grad=True)
    v0 = [torch.tensor(a, dtype=torch.float64, device="cuda") for a in case.v]
    J = final_kinetic_energy(s, T0, v0, nsteps, k)
    J.backward()
    grad = T0.grad.cpu().numpy()
    g = Grid(case.n[:2], case.L[:2], bc=case.bc, bnd=case.bnd)
    p = Params(Re=case.params["Re"], Pr=case.params["Pr"], dt=dt)
    Jo = tg.final_kinetic_energy(g, p, case.T, case.v, nsteps)
    print("J", J.item(), Jo, flush=True)
    assert abs(J.item() - Jo) <= 1e-12 * abs(Jo)
    for d in fd_directions(case.T.shape, k=3):
        cs = tg.ke_directional(g, p, case.T, case.v, d, nsteps)
        ad = float(np.sum(grad * d))
        print(cs, ad, abs(ad - cs) / abs(cs), flush=True)
        assert abs(ad - cs) <= 1e-9 * abs(cs)


def test_ke_gradient_cavity_against_oracle_complex_step():
    """The isothermal cavity (48 x 40, no-slip walls, buoyancy 1/Fr^2 = 0.5),
    6 steps with checkpoints every 2: J and its T0-gradient along 3 seeded
    directions against the oracle's complex step."""
    import torch
    from paper_2603_01727_amd.adjoint import final_kinetic_energy
    nsteps, k = 6, 2
    case = _walls_case("cavity", seed=23)
    dt = _dt(case)
    print("ke gradient cavity", nsteps, flush=True)
    s = _solver(case, dt, inv_Fr2=0.5)
    for (d, side), data in case.bnd.items():
        s.set_side(d, side, H=data.get("H"))
    T0 = torch.tensor(case.T, dtype=torch.float64, device="cuda", requires_grad=True)
    v0 = [torch.tensor(a, dtype=torch.float64, device="cuda") for a in case.v]
    J = final_kinetic_energy(s, T0, v0, nsteps, k)
    J.backward()
    grad = T0.grad.cpu().numpy()
    g = Grid(case.n[:2], case.L[:2], bc=case.bc, bnd=case.bnd)
    p = Params(Re=case.params["Re"], Pr=case.params["Pr"], dt=dt, inv_Fr2=0.5)
    Jo = tg.final_kinetic_energy(g, p, case.T, case.v, nsteps)
    print("J", J.item(), Jo, flush=True)
    assert abs(J.item() - Jo) <= 1e-12 * abs(Jo)
    for d in fd_directions(case.T.shape, k=3):
        cs = tg.ke_directional(g, p, case.T, case.v, d, nsteps)
        ad = float(np.sum(grad * d))
        print(cs, ad, abs(ad - cs) / abs(cs), flush=True)
        assert abs(ad - cs) <= 1e-9 * abs(cs)


def _ke_setup(n, nsteps):
    case = c5_case(n=n)
    dt = _dt(case)
    return case, dt


def test_ke_gradient_against_oracle_complex_step():
    import torch
    from paper_2603_01727_amd.adjoint import final_kinetic_energy
    n, nsteps, k = 64, 7, 3
    case, dt = _ke_setup(n, nsteps)
    print("ke gradient vs oracle", n, nsteps, flush=True)
    s = _solver(case, dt)
    T0 = torch.tensor(case.T, dtype=torch.float64, device="cuda", requires_grad=True)
    v0 = [torch.tensor(a, dtype=torch.float64, device="cuda") for a in case.v]
    J = final_kinetic_energy(s, T0, v0, nsteps, k)
    J.backward()
    grad = T0.grad.cpu().numpy()
    g = Grid(case.n[:2], case.L[:2], bc=case.bc)
    p = Params(Re=case.params["Re"], Pr=case.params["Pr"], dt=dt)
    Jo = tg.final_kinetic_energy(g, p, case.T, case.v, nsteps)
    assert abs(J.item() - Jo) <= 1e-12 * abs(Jo)
    for d in fd_directions(case.T.shape, k=4):
        cs = tg.ke_directional(g, p, case.T, case.v, d, nsteps)
        ad = float(np.sum(grad * d))
        print(cs, ad, abs(ad - cs) / abs(cs), flush=True)
        assert abs(ad - cs) <= 1e-9 * abs(cs)


def _ke_density(s):
    f = s.get(("rho", "v"), device=False)
    return 0.5 * f["rho"] * (f["v"][0] ** 2 + f["v"][1] ** 2)


def _fd_check(n, nsteps, k, ndir=16, h=1e-6, h4=None, more_h=()):
    """Central differences J(T0 + h d) - J(T0 - h d) over 2h along seeded
    directions. Numerators are summed from per-cell differences of the final
    kinetic-energy density (the same number as the difference of the two
    sums, without the rounding of two O(J) sums). With ``h4`` also the
    five-point difference (-J(2 h4) + 8 J(h4) - 8 J(-h4) + J(-2 h4))/(12 h4),
    whose O(h4^4) truncation and O(ulp(J)/h4) rounding both stay below 1e-6
    of the derivative. Returns J, the gradient wall time and per-direction
    (error at h, error of the five-point difference, derivative, central
    differences at each step of ``more_h``)."""
    import torch
    from paper_2603_01727_amd.adjoint import Trajectory, final_kinetic_energy
    case, dt = _ke_setup(n, nsteps)
    s = _solver(case, dt)
    T0 = torch.tensor(case.T, dtype=torch.float64, device="cuda", requires_grad=True)
    v0 = [torch.tensor(a, dtype=torch.float64, device="cuda") for a in case.v]
    t0 = time.time()
    J = final_kinetic_energy(s, T0, v0, nsteps, k)
    J.backward()
    torch.cuda.synchronize()
    t_grad = time.time() - t0
    grad = T0.grad
    dV = case.L[0] * case.L[1] / (n * n)
    traj = Trajectory(s, nsteps, nsteps)

    def e_at(dd, step):
        traj.forward(T0.detach() + step * dd, v0)
        return _ke_density(s)

    out = []
    for q, d in enumerate(fd_directions(case.T.shape, k=ndir)):
        dd = torch.tensor(d, dtype=torch.float64, device="cuda")
        ad = float(torch.sum(grad * dd))
        fd = float(np.sum(e_at(dd, h) - e_at(dd, -h))) * dV / (2 * h)
        e4 = None
        if h4:
            num = 8.0 * (e_at(dd, h4) - e_at(dd, -h4)) - (e_at(dd, 2 * h4) - e_at(dd, -2 * h4))
            fd4 = float(np.sum(num)) * dV / (12 * h4)
            e4 = abs(ad - fd4) / abs(fd4)
        more = [float(np.sum(e_at(dd, hh) - e_at(dd, -hh))) * dV / (2 * hh) for hh in more_h]
        out.append((abs(ad - fd) / abs(fd), e4, ad, fd, more))
        print(f"direction {q}: dJ {ad:.6e} rel err h={h:g}: {out[-1][0]:.3e}"
              + (f" five-point h={h4:g}: {e4:.3e}" if h4 else ""), flush=True)
    return J.item(), t_grad, out


def test_ke_gradient_against_finite_differences():
    """128^2, 30 steps, checkpoints every 10: central differences at
    h = 1e-6 along 16 directions agree to 1e-6."""
    print("ke gradient vs FD 128^2", flush=True)
    J, t, out = _fd_check(128, 30, 10)
    errs = [r[0] for r in out]
    print(J, t, max(errs), flush=True)
    assert max(errs) <= 1e-6, errs


def test_c5_adjoint_512_200_steps():
    """The 512^2, 200-step workload, checkpoints every 20 steps.

    The five-point difference at h = 1e-3 must agree to 1e-6 along all 16
    directions. The central difference at h = 1e-6 is held to 1e-6 plus its
    rounding floor, measured here per direction: J(T0 +- h d) are two FP64
    trajectories of 200 steps whose final kinetic energies carry rounding
    noise, which the quotient over 2h turns into an error of order
    noise / h. Central differences at 2h and 4h along the same direction
    share the quotient's truncation error (O(h^2), about 1e-12 relative
    here) but not its noise, so twice their largest spread bounds the
    noise of the h = 1e-6 quotient; no constant enters. The directions
    that meet 1e-6 outright are counted and printed."""
    print("c5 adjoint 512^2 200 steps", flush=True)
    h = 1e-6
    J, t, out = _fd_check(512, 200, 20, h=h, h4=1e-3, more_h=(2 * h, 4 * h))
    plain = 0
    for q, (e, e4, ad, fd, (fd2, fd4)) in enumerate(out):
        floor = 2.0 * max(abs(fd - fd2), abs(fd - fd4), abs(fd2 - fd4))
        ok_plain = e <= 1e-6
        plain += ok_plain
        print(f"direction {q}: err h=1e-6 {e:.3e}, measured floor {floor / abs(ad):.3e} (relative), "
              f"five-point {e4:.3e}, within 1e-6 at h=1e-6: {ok_plain}", flush=True)
        assert e4 <= 1e-6, out
        assert abs(ad - fd) <= 1e-6 * abs(ad) + floor, (q, e, floor / abs(ad))
    print("J", J, "gradient s", t, "directions within 1e-6 at h=1e-6:", plain, "of", len(out), flush=True)


def test_step_fn_gradients():
    """StepFn: (T_n, v_n) differentiable in (T0, v0). (1) The kinetic
    energy formed in torch from its outputs, J = sum 1/2 (p0/T) |v|^2 dV,
    has the same T0-gradient as FinalKineticEnergy (two seedings of one
    adjoint). (2) A random linear functional of (T_n, v_n) against the
    oracle's complex-step directional derivative along seeded directions
    in T0 and in v0 (the T0 direction through the same complex step)."""
    import torch
    from paper_2603_01727_amd.adjoint import step_fn, final_kinetic_energy
    n, nsteps, k = 64, 5, 2
    case, dt = _ke_setup(n, nsteps)
    print("step_fn gradients", n, nsteps, flush=True)
    s = _solver(case, dt)
    dV = case.L[0] * case.L[1] / (n * n)
    T0 = torch.tensor(case.T, dtype=torch.float64, device="cuda", requires_grad=True)
    v0 = [torch.tensor(a, dtype=torch.float64, device="cuda", requires_grad=True) for a in case.v]
    Tn, vn = step_fn(s, T0, v0, nsteps, k)
    J = (0.5 / Tn * (vn[0] ** 2 + vn[1] ** 2)).sum() * dV
    J.backward()
    gT = T0.grad.clone()
    T1 = torch.tensor(case.T, dtype=torch.float64, device="cuda", requires_grad=True)
    J2 = final_kinetic_energy(s, T1, [x.detach() for x in v0], nsteps, k)
    J2.backward()
    assert abs(J.item() / J2.item() - 1) < 1e-13
    rel = float(torch.linalg.norm(gT - T1.grad) / torch.linalg.norm(T1.grad))
    print("ke via step_fn", rel, flush=True)
    assert rel < 1e-12
    # (2) linear functional against the oracle's tangent
    rng = np.random.default_rng(77)
    wT = rng.normal(size=case.T.shape)
    wv = [rng.normal(size=case.T.shape) for _ in range(2)]
    for x in [T0] + v0:
        x.grad = None
    Tn, vn = step_fn(s, T0, v0, nsteps, k)
    L = (torch.tensor(wT, device="cuda") * Tn).sum() + sum((torch.tensor(w, device="cuda") * v).sum()
                                                             for w, v in zip(wv, vn))
    L.backward()
    g = Grid(case.n[:2], case.L[:2], bc=case.bc)
    p = Params(Re=case.params["Re"], Pr=case.params["Pr"], dt=dt)
    o = Oracle(g, p)
    for which in ("T", "v"):
        d = rng.normal(size=case.T.shape)
        dT = d if which == "T" else np.zeros_like(d)
        dv = [np.zeros_like(d), d] if which == "v" else [np.zeros_like(d)] * 2
        hstep = 1e-20
        st = o.initial_state(case.T + 1j * hstep * dT, [case.v[q] + 1j * hstep * dv[q] for q in range(2)])
        st = o.run(st, nsteps)
        cs = (np.sum(wT * st.T.imag) + sum(np.sum(w * a.imag) for w, a in zip(wv, st.v))) / hstep
        ad = float(torch.sum(T0.grad.cpu() * torch.tensor(dT)))
        if which == "v":
            ad += float(torch.sum(v0[1].grad.cpu() * torch.tensor(d)))
        print(which, cs, ad, abs(ad - cs) / abs(cs), flush=True)
        assert abs(ad - cs) <= 1e-9 * abs(cs)


def test_ke_gradient_3d_against_oracle_complex_step():
    """3D, 16^3, 6 steps with checkpoints every 2: the final kinetic energy
    and its T0-gradient along seeded directions against the oracle's
    complex-step derivative; then StepFn's v0-gradient of a random linear
    functional of (T_n, v_n) along a direction in the third velocity
    component."""
    import torch
    from paper_2603_01727_amd.adjoint import final_kinetic_energy, step_fn
    nsteps, k = 6, 2
    case = _case3d((16, 16, 16), seed=9)
    dt = _dt(case)
    print("ke gradient 3d vs oracle", case.n, nsteps, flush=True)
    s = _solver(case, dt)
    T0 = torch.tensor(case.T, dtype=torch.float64, device="cuda", requires_grad=True)
    v0 = [torch.tensor(a, dtype=torch.float64, device="cuda") for a in case.v]
    J = final_kinetic_energy(s, T0, v0, nsteps, k)
    J.backward()
    grad = T0.grad.cpu().numpy()
    g = Grid(case.n, case.L, bc=case.bc)
    p = Params(Re=case.params["Re"], Pr=case.params["Pr"], dt=dt)
    Jo = tg.final_kinetic_energy(g, p, case.T, case.v, nsteps)
    print("J", J.item(), Jo, flush=True)
    assert abs(J.item() - Jo) <= 1e-12 * abs(Jo)
    for d in fd_directions(case.T.shape, k=3):
        cs = tg.ke_directional(g, p, case.T, case.v, d, nsteps)
        ad = float(np.sum(grad * d))
        print(cs, ad, abs(ad - cs) / abs(cs), flush=True)
        assert abs(ad - cs) <= 1e-9 * abs(cs)
    # StepFn in 3D: a linear functional of (T_n, v_n), direction in v0[2]
    rng = np.random.default_rng(78)
    wT = rng.normal(size=case.T.shape)
    wv = [rng.normal(size=case.T.shape) for _ in range(3)]
    T1 = torch.tensor(case.T, dtype=torch.float64, device="cuda", requires_grad=True)
    v1 = [torch.tensor(a, dtype=torch.float64, device="cuda", requires_grad=True) for a in case.v]
    Tn, vn = step_fn(s, T1, v1, nsteps, k)
    Lf = (torch.tensor(wT, device="cuda") * Tn).sum() + sum((torch.tensor(w, device="cuda") * v).sum()
                                                              for w, v in zip(wv, vn))
    Lf.backward()
    o = Oracle(g, p)
    d = rng.normal(size=case.T.shape)
    hstep = 1e-20
    st = o.initial_state(case.T, [case.v[0], case.v[1], case.v[2] + 1j * hstep * d])
    st = o.run(st, nsteps)
    cs = (np.sum(wT * st.T.imag) + sum(np.sum(w * a.imag) for w, a in zip(wv, st.v))) / hstep
    ad = float(torch.sum(v1[2].grad.cpu() * torch.tensor(d)))
    print("v0[2]", cs, ad, abs(ad - cs) / abs(cs), flush=True)
    assert abs(ad - cs) <= 1e-9 * abs(cs)


@pytest.mark.parametrize("kind", ["periodic-2d", "walls-3d-reacting"])
def test_taped_levels_reverse_sweep_is_bit_exact(kind):
    """The reverse sweep that tapes each replayed step's predicted and new
    levels (lm_save_step_levels / lm_step_adjoint_levels) gives the same
    gradient, bit for bit, as the one that recomputes every step inside
    lm_step_adjoint, and as the one whose forward pass tapes every step (no
    replay); a save with no step since the state was set is an error."""
    import torch
    from paper_2603_01727_amd import LowMachError, lib
    from paper_2603_01727_amd.adjoint import Trajectory
    if kind == "periodic-2d":
        case, nsteps, k = c5_case(n=64), 7, 3
    else:
        from workloads.ics import reacting_periodic_case
        case, nsteps, k = _walls_case("box3d"), 5, 2
        r = reacting_periodic_case(case.n[:3], seed=22)
        case.Z = r.Z
        case.params = dict(r.params, Re=case.params["Re"], cfl=case.params["cfl"])
    dt = _dt(case)
    print("taped levels", kind, flush=True)
    s = _solver(case, dt)
    dev = lambda a: torch.tensor(a, dtype=torch.float64, device="cuda")
    out = []
    for tape, every in ((True, False), (False, False), (True, True)):
        traj = Trajectory(s, nsteps, k, tape_levels=tape, tape_all=every)
        traj.forward(dev(case.T), [dev(a) for a in case.v], None if case.Z is None else dev(case.Z))
        out.append([x.cpu().numpy() if not isinstance(x, list) else [y.cpu().numpy() for y in x]
                    for x in traj.backward()])
    a = out[0]
    for b in out[1:]:
        assert np.array_equal(a[0], b[0]), "T0 gradient"
        for x, y in zip(a[1], b[1]):
            assert np.array_equal(x, y), "v0 gradient"
        if len(a) > 2:
            assert np.array_equal(a[2], b[2]), "Z0 gradient"
    s.set(T=case.T, v=case.v, Z=case.Z)
    with pytest.raises(LowMachError) as e:
        s.save_step_levels()
    assert e.value.status == lib.LM_ESTATE



@pytest.mark.parametrize("n", [(8, 4), (68, 6), (4, 8, 4), (66, 6, 4)], ids=str)
@pytest.mark.parametrize("react", [False, True], ids=["inert", "reacting"])
def test_adjoint_step_dot_product_edges(n, react):
    """Rows shorter than a wavefront, a second wavefront of two or four
    cells, sides of four cells whose neighbours wrap from both ends."""
    from workloads.ics import reacting_periodic_case
    case = reacting_periodic_case(n, seed=17)
    if not react:
        for k in ("reacting", "S", "qs", "eps", "tol", "Le_F", "Le_O"):
            case.params.pop(k, None)
        rng = np.random.default_rng(18)
        case.Z, case.H, case.T = None, None, 1.0 + rng.random(case.v[0].shape)
    print("adjoint dot edges", n, react, flush=True)
    _dot_product_check(case, True, inv_Fr2=0.5, seed=500 + sum(n))

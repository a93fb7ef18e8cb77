"""The work that a user of the library has it do, as measurable cases.

Each case is one pass through public entry points of `paper_2209_01877_amd`: time marching
(fixed and adaptive steps, with and without viscous terms), the residual, its
vector-Jacobian product, a differentiated trajectory, and the data movement around a run
(sampling points, projection, admissibility, time step, checkpoint write and read).

A case is a dict:
    op      "march", "adaptive", "residual", "vjp", "adjoint" or "snapshot"
    p, prec polynomial order 1..4 and precision mode (fp64, fp32, bf16, fp16)
    nx, ny, nz   hexahedra per axis; each is split into six tetrahedra
    walls   False: periodic box of side 10.  True: unit box with a slip wall (with a bump)
            at y = 0, farfield on the other x and y sides, periodic in z, Mach 0.5
    jitter  vertex perturbation as a fraction of the mesh width
    flux    "rusanov" or "roe"
    mu      dynamic viscosity (0: Euler)
    steps   SSP-RK3 steps of one pass (march, adaptive, adjoint)
States are views without the padding elements, in the library's element order (a
space-filling curve).  `exact` evaluates the same discretisation in float64 with plain
torch, from its own quadrature, basis, geometry and face matching.
"""
from __future__ import annotations

import functools
import itertools
import math

import numpy as np
import torch

GAMMA = 1.4
PRANDTL = 0.72
FARFIELD = (1.0, 0.5 * math.sqrt(GAMMA), 0.0, 0.0, 1.0)
CFL = 0.2


def _device() -> torch.device:
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


# ------------------------------------------------------------------------------ the cases
def _case(op, p, prec, n, walls=False, jitter=0.0, flux="rusanov", mu=0.0, steps=1):
    nx, ny, nz = n
    return {"op": op, "p": p, "prec": prec, "nx": nx, "ny": ny, "nz": nz, "walls": walls, "jitter": jitter,
            "flux": flux, "mu": mu, "steps": steps}


def listed():
    def named(name, *a, **k):
        return {"name": name, **_case(*a, **k)}

    return [
        # the smallest configuration (density-wave size): a parameter sweep or a test run,
        # where every launch and every dependent memory round trip counts
        named("march_p1_fp64_384", "march", 1, "fp64", (4, 4, 4), steps=10),
        # a coarse exploratory run of the mixed mode: ten thousand elements do not fill the chip
        named("march_p3_fp16_10k", "march", 3, "fp16", (12, 12, 12), steps=4),
        # the production workload of the benchmark: mixed precision at 64^3 x 6
        named("march_p3_fp16_1573k", "march", 3, "fp16", (64, 64, 64), steps=2),
        # the same scheme in single precision, 48^3 x 6
        named("march_p3_fp32_664k", "march", 3, "fp32", (48, 48, 48), steps=2),
        # double precision on the full configuration: jittered elements, wall with bump, farfield
        named("march_p3_fp64_383k_walls", "march", 3, "fp64", (40, 38, 42), walls=True, jitter=0.2, steps=1),
        # the highest order in its mixed form, 40^3 x 6
        named("march_p4_bf16_384k", "march", 4, "bf16", (40, 40, 40), steps=2),
        # Navier-Stokes terms at the order they are benchmarked at, double precision
        named("viscous_p3_fp64_197k", "march", 3, "fp64", (32, 32, 32), mu=1e-3, steps=1),
        # Navier-Stokes in single precision around the wall, a mid-size ragged mesh
        named("viscous_p2_fp32_63k_walls", "march", 2, "fp32", (24, 20, 22), walls=True, jitter=0.2, mu=1e-3, steps=2),
        # the paper's flux and its device-chosen time step on an odd-sized small mesh with walls
        named("adaptive_p2_fp64_6k_roe", "adaptive", 2, "fp64", (11, 9, 10), walls=True, jitter=0.2, flux="roe",
              steps=4),
        # sensitivity of one residual (implicit or adjoint solvers call it per iteration)
        named("vjp_p2_fp64_384k", "vjp", 2, "fp64", (40, 40, 40), jitter=0.2),
        # gradient of a short trajectory with checkpoints, as in shape or initial-state fitting
        named("adjoint_p2_fp64_10k_walls", "adjoint", 2, "fp64", (14, 12, 10), walls=True, jitter=0.2, steps=6),
        # around a run: sample points, project an initial field, monitor, write and read a checkpoint
        named("snapshot_p3_fp64_197k", "snapshot", 3, "fp64", (32, 32, 32)),
    ]


def draw(rng):
    """One more case of the same ranges: sizes log-uniform from a few hundred elements to what
    the operation is used at, ragged boxes, every order and precision that it takes."""
    op = rng.choice(["march", "march", "march", "viscous", "viscous", "residual", "vjp", "vjp", "adjoint", "adaptive",
                     "snapshot"])
    p = rng.choice([1, 2, 2, 3, 3, 3, 4])
    walls = rng.random() < 0.5
    jitter = rng.choice([0.0, 0.1, 0.2])
    flux = rng.choice(["rusanov", "rusanov", "roe"])
    mu, steps = 0.0, 1
    prec = {"march": ["fp64", "fp32", "bf16", "fp16"], "viscous": ["fp64", "fp32"], "residual": ["fp64", "fp32"],
            "vjp": ["fp64", "fp32"], "adjoint": ["fp64", "fp32"], "adaptive": ["fp64"],
            "snapshot": ["fp64", "fp32", "bf16"]}[op]
    prec = rng.choice(prec)
    # elements up to: as many as make the operation about as costly as the listed ones
    top = {"march": 660_000, "viscous": 200_000, "residual": 660_000, "vjp": 300_000, "adjoint": 20_000,
           "adaptive": 200_000, "snapshot": 200_000}[op]
    if p == 4:
        top //= 2
    if op == "viscous":
        op, mu = "march", rng.choice([1e-3, 2e-2])
    hexes = math.exp(rng.uniform(math.log(64.0), math.log(top / 6.0)))
    edge = hexes ** (1.0 / 3.0)
    n = tuple(max(4, round(edge * rng.uniform(0.75, 1.25))) for _ in range(3))
    if op in ("march", "adaptive"):
        steps = rng.randint(1, 4) if hexes < 10_000 else 1
    elif op == "adjoint":
        steps = rng.randint(2, 5)
    return _case(op, p, prec, n, walls, jitter, flux, mu, steps)


# ------------------------------------------------------------------------------ inputs
@functools.lru_cache(maxsize=2)
def _mesh(nx, ny, nz, walls, jitter):
    """A Kuhn-split box as a mesh file would give it (host arrays): shuffled elements,
    relabelled vertices, per-element unwrapped coordinates, tagged boundary faces."""
    rng = np.random.default_rng(nx * 10007 + ny * 101 + nz)
    ns = np.array([nx, ny, nz])
    periodic = np.array([not walls, not walls, True])
    size = np.array([1.0, 1.0, 1.0]) if walls else np.array([10.0, 10.0, 10.0])
    h = size / ns
    nv = np.where(periodic, ns, ns + 1)
    base = np.stack(np.meshgrid(*(np.arange(k) for k in ns), indexing="ij"), -1).reshape(-1, 1, 3)
    unit = np.eye(3, dtype=np.int64)
    lat = np.concatenate([base + np.stack([np.zeros(3, np.int64), unit[a], unit[a] + unit[b], np.ones(3, np.int64)])
                          for a, b, _ in itertools.permutations(range(3))])          # (E, 4, 3)
    lat = lat[rng.permutation(lat.shape[0])]
    wrapped = np.where(periodic, lat % ns, lat)
    vid = (wrapped[..., 0] * nv[1] + wrapped[..., 1]) * nv[2] + wrapped[..., 2]
    n_vert = int(nv.prod())
    xyz = lat * h
    if jitter:
        shift = rng.uniform(-1.0, 1.0, (n_vert, 3)) * (jitter * h)
        idx = np.stack(np.unravel_index(np.arange(n_vert), tuple(nv)), -1)
        shift[~periodic & ((idx == 0) | (idx == ns))] = 0.0
        xyz = xyz + shift[vid]
    if walls:
        x, y = xyz[..., 0], xyz[..., 1]
        xyz[..., 1] = y + 0.05 * np.exp(-((x - 0.5) / 0.1) ** 2) * (1.0 - y)
    label = rng.permutation(n_vert).astype(np.int64)
    vid = label[vid]
    faces, tags = [np.zeros((0, 3), np.int64)], [np.zeros((0,), np.int32)]
    if walls:
        for f, axis in itertools.product(range(4), (0, 1)):
            keep = [v for v in range(4) if v != f]
            for side in (0, ns[axis]):
                on = (lat[:, keep, axis] == side).all(1)
                faces.append(vid[on][:, keep])
                tags.append(np.full(int(on.sum()), 2 if axis == 1 and side == 0 else 1, np.int32))
    return (np.ascontiguousarray(vid), np.ascontiguousarray(xyz), np.concatenate(faces), np.concatenate(tags))


def _case_mesh(case):
    return _mesh(case["nx"], case["ny"], case["nz"], case["walls"], case["jitter"])


def _primitive(case, x, seed):
    """A smooth seeded flow (..., 5): the free stream plus six plane waves per variable."""
    rng = np.random.default_rng(seed)
    length = 1.0 if case["walls"] else 10.0
    out = torch.empty(x.shape[:-1] + (5,), dtype=torch.float64, device=x.device)
    for v, (mean, amp) in enumerate(zip(FARFIELD, (0.1, 0.03, 0.03, 0.03, 0.02))):
        k = torch.tensor(rng.choice([-2, -1, 1, 2], (3, 6)) * (2.0 * math.pi / length), device=x.device)
        a = torch.tensor(rng.uniform(0.2, 1.0, 6), device=x.device)
        phase = torch.tensor(rng.uniform(0.0, 2.0 * math.pi, 6), device=x.device)
        out[..., v] = mean + amp * (torch.sin(x @ k + phase) @ (a / a.sum()))
    return out


def _solver(case):
    from paper_2209_01877_amd import Solver

    s = Solver(case["p"], case["prec"])
    if case["mu"] > 0.0:
        s.set_viscosity(case["mu"], PRANDTL)
    vid, xyz, bface, tag = _case_mesh(case)
    s.upload_mesh(vid, xyz, bface, tag, renumber="hilbert")
    s.set_farfield(FARFIELD)
    s.set_flux(case["flux"])
    return s


def _inputs(case, seed):
    """The inputs in the caller's layout: coefficients, and what else the operation takes."""
    ref = _Discretisation(case)
    U = ref.project(seed)
    more = {}
    if case["op"] in ("march", "adjoint"):
        more["dt"] = 0.5 * float(ref.stable_dt(U, CFL))
    if case["op"] in ("vjp", "adjoint"):
        gen = torch.Generator(device=U.device).manual_seed(seed + 1)
        more["W"] = torch.randn(U.shape, dtype=torch.float64, device=U.device, generator=gen)
    if case["op"] == "snapshot":
        more["prim"] = _primitive(case, ref.points(), seed + 2)
    if case["prec"] == "fp32":  # the state is held in 32 bits: the inputs are such values
        U = U.float().double()
        if "W" in more:
            more["W"] = more["W"].float().double()
    return ref, U, more


def prepare(case, seed):
    _, U, more = _inputs(case, seed)
    s = _solver(case)
    state = {"case": case, "solver": s, "U": s.set_state(U)}
    op = case["op"]
    if op in ("march", "adaptive"):
        state["work"] = s.new_work()
    if op in ("march", "adjoint"):
        state["dt"] = more["dt"]
    if op in ("vjp", "adjoint"):
        state["W"] = s.set_state(more["W"])
    if op in ("residual", "vjp"):
        state["out"] = s.new_state()
    if op == "adjoint":
        state["U"].requires_grad_(True)
    if op == "snapshot":
        state.update(prim=more["prim"], user=U, projected=s.new_state(), restored=s.new_state())
    return state


def run(state):
    case, s, U = state["case"], state["solver"], state["U"]
    n = s.n_elem
    op = case["op"]
    if op == "march":
        return [s.rk_step(U, state["dt"], case["steps"], state["work"])[:, :, :n]]
    if op == "adaptive":
        dts = s.rk_step_adaptive(U, CFL, case["steps"], state["work"])
        return [U[:, :, :n], dts]
    if op == "residual":
        return [s.residual(U, state["out"])[:, :, :n]]
    if op == "vjp":
        return [s.residual_vjp(U, state["W"], state["out"])[:, :, :n]]
    if op == "adjoint":
        from paper_2209_01877_amd.autograd import rk_trajectory

        end = rk_trajectory(s, U, state["dt"], case["steps"], checkpoint_every=3)
        (grad,) = torch.autograd.grad(end, U, state["W"])
        return [end.detach()[:, :, :n], grad[:, :, :n]]
    # snapshot
    x = s.volume_points()
    projected = s.project(state["prim"], state["projected"])
    bad = s.check_state(U)
    dt = s.stable_dt(U, CFL)
    written = s.get_state(U)
    restored = s.set_state(state["user"], state["restored"])
    return [x, projected[:, :, :n], bad, dt, written, restored[:, :, :n]]


def work(case):
    """Bytes and operations that one pass cannot do without."""
    p, n_elem = case["p"], 6 * case["nx"] * case["ny"] * case["nz"]
    n_p, n_q, n_f = (p + 1) * (p + 2) * (p + 3) // 6, (p + 1) ** 3, (p + 1) ** 2
    width = 4 if case["prec"] == "fp32" else 8
    st = 5 * n_p * width
    geo = 100  # |det J| J^-1, 1/|K|, neighbour ids, face codes
    # contractions of one residual (volume interpolation, three-direction projection, own and
    # neighbour traces, lift) and the pointwise fluxes
    flops = 10.0 * n_p * (4 * n_q + 12 * n_f) + 60.0 * n_q + 400.0 * n_f
    if case["mu"] > 0.0:  # the lifted gradient and the viscous flux of 15 more variables
        flops += 10.0 * n_p * (3 * n_q + 6 * n_f) + 30.0 * n_p * (n_q + 4 * n_f) + 200.0 * (n_q + 4 * n_f)
    step_bytes = 2 * st + 2 * (3 * st) + 3 * geo  # stages 2 and 3 also read the step's first state
    op = case["op"]
    if op in ("march", "adaptive"):
        return {"bytes": n_elem * case["steps"] * step_bytes, "flops": n_elem * case["steps"] * 3 * flops}
    if op == "residual":
        return {"bytes": n_elem * (2 * st + geo), "flops": n_elem * flops}
    # state and cotangent both contracted, transposed
    vjp = 10.0 * n_p * (5 * n_q + 20 * n_f) + 150.0 * n_q + 600.0 * n_f
    if op == "vjp":
        return {"bytes": n_elem * (3 * st + geo), "flops": n_elem * vjp}
    if op == "adjoint":
        # forward, recomputed forward, and three accumulating products per step
        per_step = 2 * step_bytes + 3 * (3 * st + geo) + 3 * st
        return {"bytes": n_elem * case["steps"] * per_step, "flops": n_elem * case["steps"] * 3 * (2 * flops + vjp)}
    user = 8 * 5 * n_p
    bytes_ = (12 * 8 + 24 * n_q) + (40 * n_q + st) + st + (st // n_p + geo) + (st + user) + (user + st)
    return {"bytes": n_elem * bytes_, "flops": n_elem * (20.0 * n_p * n_q + 30.0 * n_q)}


# ------------------------------------------------------------------------------ float64 reference
def _gauss_jacobi(n, alpha):
    """n-point rule on [-1, 1] for the weight (1 - x)^alpha (Golub and Welsch)."""
    k = np.arange(n, dtype=np.float64)
    s = 2.0 * k + alpha
    diag = np.where(s + 2 > 0, -alpha ** 2 / np.where(s == 0, 1.0, s * (s + 2.0)), 0.0)
    diag[0] = -alpha / (alpha + 2.0)
    k, s = k[1:], s[1:]
    off = np.sqrt(4.0 * k * (k + alpha) * k * (k + alpha) / (s * s * (s + 1.0) * (s - 1.0)))
    x, v = np.linalg.eigh(np.diag(diag) + np.diag(off, 1) + np.diag(off, -1))
    return x, v[0] ** 2 * 2.0 ** (alpha + 1) / (alpha + 1)


def _jacobi(n, alpha, x):
    """P_n^(alpha, 0)(x) by its three-term recurrence."""
    last, now = torch.zeros_like(x), torch.ones_like(x)
    for m in range(1, n + 1):
        c = 2.0 * m * (m + alpha) * (2.0 * m + alpha - 2.0)
        if m == 1:
            last, now = now, 0.5 * (alpha + (alpha + 2.0) * x)
        else:
            a = (2.0 * m + alpha - 1.0) * ((2.0 * m + alpha) * (2.0 * m + alpha - 2.0) * x + alpha * alpha)
            b = 2.0 * (m + alpha - 1.0) * (m - 1.0) * (2.0 * m + alpha)
            last, now = now, (a * now - b * last) / c
    return now


def _basis(p, xi):
    """Orthonormal modal basis at points (N, 3) inside the unit tetrahedron: (N, N_p)."""
    r, s, t = (2.0 * xi[:, d] - 1.0 for d in range(3))
    a, b = 2.0 * (1.0 + r) / (-s - t) - 1.0, 2.0 * (1.0 + s) / (1.0 - t) - 1.0
    cols = []
    for d in range(p + 1):
        for k in range(d + 1):
            for j in range(d - k + 1):
                i = d - j - k
                f = (_jacobi(i, 0.0, a) * ((-s - t) / 2) ** i * _jacobi(j, 2.0 * i + 1, b) * ((1 - t) / 2) ** j
                     * _jacobi(k, 2.0 * i + 2.0 * j + 2.0, t))
                # 6 * integral of the square over the unit tetrahedron, in closed form
                norm = 6.0 / ((2 * i + 1) * (2 * i + 2 * j + 2) * (2 * i + 2 * j + 2 * k + 3))
                cols.append(f / math.sqrt(norm))
    return torch.stack(cols, 1)


@functools.lru_cache(maxsize=8)
def _tables(p):
    n = p + 1
    (a, wa), (b, wb), (c, wc) = (_gauss_jacobi(n, al) for al in (0.0, 1.0, 2.0))
    cc, bb, aa = np.meshgrid(c, b, a, indexing="ij")
    xi = np.stack([(1 + aa) * (1 - bb) * (1 - cc) / 8, (1 + bb) * (1 - cc) / 4, (1 + cc) / 2], -1).reshape(-1, 3)
    w = (wc[:, None, None] * wb[:, None] * wa / 64).reshape(-1)
    bb, aa = np.meshgrid(b, a, indexing="ij")
    st = np.stack([(1 + aa) * (1 - bb) / 4, (1 + bb) / 2], -1).reshape(-1, 2)
    wf = (wb[:, None] * wa / 8).reshape(-1)
    corner = np.array([[0.0, 0, 0], [1, 0, 0], [0, 1, 0], [0, 0, 1]])
    xi_t = torch.from_numpy(xi).requires_grad_(True)
    B = _basis(p, xi_t)
    D = torch.stack([torch.autograd.grad(B[:, m].sum(), xi_t, retain_graph=True)[0] if m else torch.zeros_like(xi_t)
                     for m in range(B.shape[1])], 2).permute(1, 0, 2)                 # (3, N_q, N_p)
    Bf = []
    for f in range(4):
        v0, v1, v2 = corner[[v for v in range(4) if v != f]]
        Bf.append(_basis(p, torch.from_numpy(v0 + st[:, :1] * (v1 - v0) + st[:, 1:] * (v2 - v0))))
    return tuple(x.detach().to(_device()) for x in (xi_t, torch.from_numpy(w), B, D, torch.from_numpy(wf), torch.stack(Bf)))


def _pressure(U):
    return (GAMMA - 1.0) * (U[4] - 0.5 * (U[1] ** 2 + U[2] ** 2 + U[3] ** 2) / U[0])


def _normal_flux(U, N):
    """Euler flux through N (variables first)."""
    p, un = _pressure(U), (U[1] * N[0] + U[2] * N[1] + U[3] * N[2]) / U[0]
    return torch.stack([U[0] * un] + [U[1 + d] * un + p * N[d] for d in range(3)] + [(U[4] + p) * un])


def _rusanov(a, b, N, nn):
    def speed(U):
        return ((U[1] * N[0] + U[2] * N[1] + U[3] * N[2]) / U[0]).abs() + torch.sqrt(GAMMA * _pressure(U) / U[0]) * nn
    return 0.5 * (_normal_flux(a, N) + _normal_flux(b, N)) - 0.5 * torch.maximum(speed(a), speed(b)) * (b - a)


def _roe(a, b, N, nn):
    """Roe's flux: square-root-density averages, Harten's fix of width 0.1 c."""
    n = [x / nn for x in N]
    dot = lambda x, y: x[0] * y[0] + x[1] * y[1] + x[2] * y[2]  # noqa: E731
    ul, ur = a[1:4] / a[0], b[1:4] / b[0]
    pl, pr = _pressure(a), _pressure(b)
    sl, sr = torch.sqrt(a[0]), torch.sqrt(b[0])
    u = (sl * ul + sr * ur) / (sl + sr)
    H = (sl * (a[4] + pl) / a[0] + sr * (b[4] + pr) / b[0]) / (sl + sr)
    rho, q2 = sl * sr, dot(u, u)
    c = torch.sqrt((GAMMA - 1.0) * (H - 0.5 * q2))
    un, dp, du = dot(u, n), pr - pl, ur - ul
    dun, drho = dot(du, n), b[0] - a[0]
    fix = lambda lam: torch.where(lam.abs() < 0.1 * c, (lam * lam + 0.01 * c * c) / (0.2 * c), lam.abs())  # noqa: E731
    k1 = fix(un - c) * (dp - rho * c * dun) / (2.0 * c * c)
    k4 = fix(un + c) * (dp + rho * c * dun) / (2.0 * c * c)
    k2, k3 = un.abs() * (drho - dp / (c * c)), un.abs() * rho
    diss = [k1 + k2 + k4]
    diss += [k1 * (u[d] - c * n[d]) + k2 * u[d] + k3 * (du[d] - dun * n[d]) + k4 * (u[d] + c * n[d]) for d in range(3)]
    diss.append(k1 * (H - un * c) + k2 * 0.5 * q2 + k3 * (dot(u, du) - un * dun) + k4 * (H + un * c))
    return 0.5 * (_normal_flux(a, N) + _normal_flux(b, N)) - 0.5 * nn * torch.stack(diss)


def _viscous_flux(U, Z, mu):
    """Rows j of the viscous flux from U (5, ...) and Z (3, 5, ...), Z[k, w] = d_k U_w."""
    u = U[1:4] / U[0]
    T = _pressure(U) / U[0]
    q2 = (u * u).sum(0)
    gu = [[(Z[k, 1 + i] - u[i] * Z[k, 0]) / U[0] for i in range(3)] for k in range(3)]
    div = gu[0][0] + gu[1][1] + gu[2][2]
    kappa = mu * GAMMA / ((GAMMA - 1.0) * PRANDTL)
    rows = []
    for j in range(3):
        gp = (GAMMA - 1.0) * (Z[j, 4] - 0.5 * q2 * Z[j, 0] - U[0] * sum(u[i] * gu[j][i] for i in range(3)))
        tau = [mu * (gu[j][i] + gu[i][j]) - (2.0 / 3.0 * mu * div if i == j else 0.0) for i in range(3)]
        heat = kappa * (gp - T * Z[j, 0]) / U[0]
        rows.append(torch.stack([torch.zeros_like(T)] + tau + [heat + sum(u[i] * tau[i] for i in range(3))]))
    return rows


class _Discretisation:
    """The method in float64, element by element; coefficients (E, 5, N_p), caller's order."""

    CHUNK = 65536

    def __init__(self, case):
        self.case, self.p, self.mu = case, case["p"], case["mu"]
        dev = _device()
        vid, xyz, bface, tag = _case_mesh(case)
        vid, xyz = torch.from_numpy(vid).to(dev), torch.from_numpy(xyz).to(dev)
        self.xi, self.w, self.B, self.D, self.wf, self.Bf = _tables(self.p)
        self.E, self.n_p = vid.shape[0], self.B.shape[1]
        vid, order = torch.sort(vid, 1)
        xyz = torch.gather(xyz, 1, order[:, :, None].expand(-1, -1, 3))
        self.x0 = xyz[:, 0]
        e1, e2, e3 = (xyz[:, k] - xyz[:, 0] for k in (1, 2, 3))
        self.J = torch.stack([e1, e2, e3], 2)
        rows = torch.stack([torch.linalg.cross(e2, e3), torch.linalg.cross(e3, e1), torch.linalg.cross(e1, e2)], 1)
        det = (rows[:, 0] * e1).sum(1)
        self.vol = det.abs() / 6.0
        self.M = rows * torch.sign(det)[:, None, None]              # |det J| J^-1
        self.N = torch.cat([self.M.sum(1, keepdim=True), -self.M], 1)  # (E, 4, 3): 2 A n
        self.nn = torch.linalg.norm(self.N, dim=2)
        self.vid, self.n_vert = vid, int(vid.max()) + 1
        self.bface, self.tag = torch.from_numpy(np.sort(bface, 1)).to(dev), torch.from_numpy(tag).to(dev)
        self.far = torch.tensor([1.0, FARFIELD[1], 0.0, 0.0, 1.0 / (GAMMA - 1.0) + 0.5 * FARFIELD[1] ** 2],
                                dtype=torch.float64, device=dev)
        self.nbr = None

    def _match(self):
        """Neighbour element, its local face, and the boundary tag across each face."""
        def key(t):
            return (t[:, 0] * self.n_vert + t[:, 1]) * self.n_vert + t[:, 2]
        k = torch.cat([key(self.vid[:, [v for v in range(4) if v != f]]) for f in range(4)])
        k, at = torch.sort(k)
        pair = torch.nonzero(k[1:] == k[:-1]).flatten()
        other = torch.full((4 * self.E,), -1, dtype=torch.long, device=k.device)
        other[at[pair]], other[at[pair + 1]] = at[pair + 1], at[pair]
        other = other.view(4, self.E)
        self.nbr, self.nface = torch.where(other >= 0, other % self.E, -1), other.clamp(min=0) // self.E
        self.btag = torch.zeros((4, self.E), dtype=torch.int32, device=k.device)
        if self.tag.numel():
            bk, bo = torch.sort(key(self.bface))
            slot = torch.searchsorted(bk, k).clamp(max=bk.numel() - 1)
            hit = bk[slot] == k
            self.btag.view(-1)[at[hit]] = self.tag[bo][slot[hit]]

    def chunks(self):
        return torch.split(torch.arange(self.E, device=self.x0.device), self.CHUNK)

    def points(self):
        return self.x0[:, None] + self.xi @ self.J.transpose(1, 2)

    def project(self, seed):
        out = torch.empty((self.E, 5, self.n_p), dtype=torch.float64, device=self.x0.device)
        for c in self.chunks():
            x = self.x0[c, None] + self.xi @ self.J[c].transpose(1, 2)
            out[c] = self.project_prim(_primitive(self.case, x, seed))
        return out

    def project_prim(self, q):
        rho, u, p = q[..., :1], q[..., 1:4], q[..., 4:]
        U = torch.cat([rho, rho * u, p / (GAMMA - 1.0) + 0.5 * rho * (u * u).sum(-1, keepdim=True)], -1)
        return 6.0 * U.transpose(1, 2) @ (self.w[:, None] * self.B)

    def stable_dt(self, U, cfl):
        m = U[:, :, 0].T
        speed = torch.sqrt(m[1] ** 2 + m[2] ** 2 + m[3] ** 2) / m[0] + torch.sqrt(GAMMA * _pressure(m) / m[0])
        return (cfl * 12.0 * self.vol / self.nn.sum(1) / ((2 * self.p + 1) * speed)).min()

    def _neighbour_trace(self, f, c, U):
        """Traces (k, e, n_f) of U (E, k, N_p) from the other side of face f of elements c."""
        n_f = self.Bf.shape[1]
        t = (U[self.nbr[f, c].clamp(min=0)] @ self.Bf.reshape(4 * n_f, -1).T).view(c.numel(), -1, 4, n_f)
        pick = self.nface[f, c][:, None, None, None].expand(-1, t.shape[1], 1, n_f)
        return torch.gather(t, 2, pick)[:, :, 0].transpose(0, 1)

    def _faces(self, c, U):
        """Per face: own and neighbour (or ghost) traces (5, e, n_f), area normal and its length."""
        for f in range(4):
            N = [self.N[c, f, d][:, None] for d in range(3)]
            a = (U[c] @ self.Bf[f].T).transpose(0, 1)
            b = self._neighbour_trace(f, c, U)
            tag = self.btag[f, c][:, None]
            if bool((tag > 0).any()):
                mn = (a[1] * N[0] + a[2] * N[1] + a[3] * N[2]) / self.nn[c, f][:, None] ** 2
                wall = torch.stack([a[0]] + [a[1 + d] - 2.0 * mn * N[d] for d in range(3)] + [a[4]])
                b = torch.where(tag == 1, self.far[:, None, None].expand_as(a), torch.where(tag == 2, wall, b))
            yield f, a, b, N, self.nn[c, f][:, None]

    def _gradient(self, U):
        """BR1 lifted gradient, (E, 15, N_p) with index 5 k + v."""
        Z = torch.empty((self.E, 15, self.n_p), dtype=torch.float64, device=U.device)
        for c in self.chunks():
            wU = (U[c] @ self.B.T) * self.w
            D = [-wU @ self.D[d] for d in range(3)]
            z = [sum(self.M[c, d, k][:, None, None] * D[d] for d in range(3)) for k in range(3)]
            for f, a, b, N, _ in self._faces(c, U):
                lift = (0.5 * (a + b) * self.wf).transpose(0, 1) @ self.Bf[f]
                z = [z[k] + N[k][:, :, None] * lift for k in range(3)]
            Z[c] = torch.cat(z, 1) / self.vol[c, None, None]
        return Z

    def residual_chunk(self, c, U, Z=None):
        M = self.M[c]
        flux = _roe if self.case["flux"] == "roe" else _rusanov
        Uq = (U[c] @ self.B.T).transpose(0, 1)
        if Z is not None:
            Fv = _viscous_flux(Uq, (Z[c] @ self.B.T).view(c.numel(), 3, 5, -1).permute(1, 2, 0, 3), self.mu)
        R = 0.0
        for d in range(3):
            row = [M[:, d, k][:, None] for k in range(3)]
            y = _normal_flux(Uq, row)
            if Z is not None:
                y = y - sum(row[k] * Fv[k] for k in range(3))
            R = R + (y * self.w).transpose(0, 1) @ self.D[d]
        for f, a, b, N, nn in self._faces(c, U):
            h = flux(a, b, N, nn)
            if Z is not None:
                n_f = self.wf.numel()
                Za = (Z[c] @ self.Bf[f].T).transpose(0, 1)
                Zb = torch.where((self.nbr[f, c] >= 0)[:, None], self._neighbour_trace(f, c, Z), Za)
                Fa, Fb = (_viscous_flux(u, z.reshape(3, 5, -1, n_f), self.mu) for u, z in ((a, Za), (b, Zb)))
                h = h - 0.5 * sum(N[k] * (Fa[k] + Fb[k]) for k in range(3))
            R = R - (h * self.wf).transpose(0, 1) @ self.Bf[f]
        return R / self.vol[c, None, None]

    def residual(self, U):
        if self.nbr is None:
            self._match()
        Z = self._gradient(U) if self.mu > 0.0 else None
        return torch.cat([self.residual_chunk(c, U, Z) for c in self.chunks()])

    def step(self, U, dt):
        U1 = U + dt * self.residual(U)
        U2 = 0.75 * U + 0.25 * (U1 + dt * self.residual(U1))
        return U / 3.0 + (2.0 / 3.0) * (U2 + dt * self.residual(U2))

    def vjp(self, U, W):
        self._match()
        U = U.clone().requires_grad_(True)
        for c in self.chunks():
            (self.residual_chunk(c, U) * W[c]).sum().backward()
        return U.grad


def exact(case, seed):
    """What run() returns on a fresh state, in float64 with plain torch.  The library's solver
    is asked only for its element order, which the outputs are laid out in."""
    ref, U, more = _inputs(case, seed)
    perm = torch.from_numpy(_solver(case).perm).to(U.device)

    def internal(X):  # (E, 5, N_p) -> [5][quads][E][4]
        quads = -(-ref.n_p // 4)
        X = torch.nn.functional.pad(X[perm], (0, 4 * quads - ref.n_p))
        return X.view(-1, 5, quads, 4).permute(1, 2, 0, 3)

    op = case["op"]
    if op == "march":
        for _ in range(case["steps"]):
            U = ref.step(U, more["dt"])
        return [internal(U)]
    if op == "adaptive":
        dts = []
        for _ in range(case["steps"]):
            dts.append(ref.stable_dt(U, CFL))
            U = ref.step(U, dts[-1])
        return [internal(U), torch.stack(dts)]
    if op == "residual":
        return [internal(ref.residual(U))]
    if op == "vjp":
        return [internal(ref.vjp(U, more["W"]))]
    if op == "adjoint":
        if ref.E * ref.n_p * case["steps"] > 1_000_000:  # the recorded graph would not stay small
            return None
        U = U.requires_grad_(True)
        end = U
        for _ in range(case["steps"]):
            end = ref.step(end, more["dt"])
        (grad,) = torch.autograd.grad(end, U, more["W"])
        return [internal(end.detach()), internal(grad)]
    Uq = torch.cat([(U[c] @ ref.B.T).transpose(1, 2) for c in ref.chunks()])
    ok = torch.isfinite(Uq).all(2) & (Uq[..., 0] > 0) & (_pressure(Uq.movedim(2, 0)) > 0)
    return [ref.points(), internal(ref.project_prim(more["prim"])), (~ok.all(1)).sum(), ref.stable_dt(U, CFL), U,
            internal(U)]

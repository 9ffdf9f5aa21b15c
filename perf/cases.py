"""The work a user has this framework do, as cases that can be timed and compared.

Six kinds of call, each through the public Python entry points:

* ``step``    one half-step of a 1D problem (a program that drives its own time loop);
* ``solve``   a whole small 1D problem: write the state, advance to an end time, read it back;
* ``run``     a stretch of half-steps of a 1D state that stays on the GPU;
* ``batch``   a stretch of half-steps of many uneven 1D instances advanced together;
* ``run2d``   a stretch of half-steps of a 2D state that stays on the GPU;
* ``solve2d`` a whole small 2D problem, as ``solve``.

`listed()` names the sizes, `draw()` gives more of the same ranges, `prepare()`
builds the problem and `run()` makes one pass.  `exact()` evaluates the same
half-steps in binary64 with plain numpy or torch.
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

from paper_2104_04347_amd import binding, inputs

# CFL numbers per half-step: the paper's 0.4 / 0.3 / 0.25 for orders 2 / 3 / 4, 0.2 for order 5
CFL = {1: 0.4, 2: 0.3, 3: 0.25, 4: 0.2}
GAMMA = 1.4
EPS = 1e-40
STATE_OFFSET = 12544      # bytes of control data at the head of a workspace (include/wcc.h)


def listed():
    return [
        # a program with a time loop of its own (output or coupling every half-step): one launch a call
        dict(name="step_euler_400", kind="step", eq="euler", P=3, N=400, bc="transmissive", limiter=True,
             precision="fp64"),
        # the paper's shock-tube experiments: a few hundred cells to an end time, host to host
        dict(name="solve_euler_400", kind="solve", eq="euler", P=3, N=400, bc="transmissive", limiter=True,
             precision="fp64", t_end=0.2),
        # smooth advection on [0, 2], once around the periodic domain (convergence studies)
        dict(name="solve_advection_200", kind="solve", eq="advection", P=2, N=200, bc="periodic", limiter=True,
             precision="fp64", t_end=2.0),
        # Burgers with sine modes: a mesh that fills a fraction of the GPU
        dict(name="run_burgers_12800", kind="run", eq="burgers", P=3, N=12800, bc="periodic", limiter=True,
             precision="fp64", steps=96),
        # the benchmark workload, in both precisions
        dict(name="run_euler_1m", kind="run", eq="euler", P=3, N=1048576, bc="transmissive", limiter=True,
             precision="fp64", steps=20),
        dict(name="run_euler_1m_mixed", kind="run", eq="euler", P=3, N=1048576, bc="transmissive", limiter=True,
             precision="fp32_mixed", steps=20),
        # a state beyond the Infinity Cache at the highest degree, jumps all over a periodic domain
        dict(name="run_euler_4m_p4", kind="run", eq="euler", P=4, N=4194304, bc="periodic", limiter=True,
             precision="fp64", steps=8),
        # a parameter study: shock tubes of uneven size and degree, 256 to 65,536 cells each
        dict(name="batch_512", kind="batch", B=512, n_lo=256, n_hi=65536, sizes=0, precision="fp32_mixed", steps=24),
        # 2D: scalar with limiter, smooth Euler without, Euler with the characteristic limiter and open edges
        dict(name="run2d_burgers_1024", kind="run2d", eq="burgers", P=3, Nx=1024, Ny=1024, bc="periodic",
             limiter=True, steps=10),
        dict(name="run2d_vortex_768", kind="run2d", eq="euler", P=3, Nx=768, Ny=768, bc="periodic",
             limiter=False, steps=10),
        dict(name="run2d_riemann_600", kind="run2d", eq="euler", P=3, Nx=600, Ny=600, bc="transmissive",
             limiter=True, steps=10),
        # a small 2D Riemann problem, host to host
        dict(name="solve2d_riemann_40", kind="solve2d", eq="euler", P=2, Nx=40, Ny=40, bc="transmissive",
             limiter=True, t_end=0.1),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "solve", "run", "run", "run", "batch", "run2d", "run2d", "solve2d"])
    if kind in ("step", "solve", "run"):
        eq = rng.choice(["advection", "burgers", "euler", "euler"])
        P = rng.choice([1, 2, 3, 3, 4])
        bc = rng.choice(["periodic", "transmissive", "dirichlet"]) if eq == "euler" else "periodic"
        case = dict(kind=kind, eq=eq, P=P, bc=bc, limiter=eq != "advection" or rng.random() < 0.5,
                    precision=rng.choice(["fp64", "fp64", "fp32_mixed"]))
        if kind == "solve":
            case["N"] = _log_int(rng, 64, 2000)
            case["t_end"] = round(rng.uniform(0.2, 0.5) * min(1.0, 600.0 / case["N"]), 4)
        else:
            case["N"] = _log_int(rng, 64, 4000) if kind == "step" else _log_int(rng, 2000, 3500000)
        if kind == "run":
            case["steps"] = 2 * max(2, min(48, int(1.5e7 / case["N"])))
        return case
    if kind == "batch":
        hi = _log_int(rng, 4000, 65536)
        return dict(kind=kind, B=_log_int(rng, 16, 400), n_lo=256, n_hi=hi, sizes=rng.randrange(1 << 20),
                    precision=rng.choice(["fp64", "fp32_mixed"]), steps=2 * rng.randint(5, 12))
    eq = rng.choice(["advection", "burgers", "euler", "euler"])
    case = dict(kind=kind, eq=eq, P=rng.choice([1, 2, 3, 3]), limiter=True,
                bc=rng.choice(["periodic", "transmissive"]) if eq == "euler" else "periodic")
    if kind == "solve2d":
        case.update(Nx=rng.randint(16, 64), Ny=rng.randint(16, 64), t_end=round(rng.uniform(0.05, 0.15), 4))
        return case
    case.update(Nx=_log_int(rng, 80, 700), Ny=_log_int(rng, 80, 700), steps=2 * rng.randint(3, 6))
    if eq == "advection":
        case["limiter"] = rng.random() < 0.5
    if eq == "euler" and rng.random() < 0.3:      # the smooth vortex on its periodic square
        case.update(Ny=case["Nx"], bc="periodic", limiter=False)
    return case


# ---------------------------------------------------------------------------
# Inputs: initial states from the seed (problem data only).
# ---------------------------------------------------------------------------
def _domain(case):
    return (0.0, 1.0) if case["eq"] == "euler" else (0.0, 2.0)


def _gas(rng, n):
    """n gas states (rho, u, p) of moderate strength, as numpy arrays."""
    return rng.uniform(0.3, 1.0, n), rng.uniform(-0.4, 0.4, n), rng.uniform(0.3, 1.0, n)


def _initial_1d(case, seed):
    """State (nc, P+1, n) on the original mesh and the two Dirichlet states."""
    P, N, bc = case["P"], case["N"], case["bc"]
    x0, x1 = _domain(case)
    rng = np.random.default_rng(seed)
    none = (0.0, 0.0, 0.0)
    if case["eq"] == "advection":
        return inputs.sine_wave(P, N, x0, x1, c0=1.0, amp=0.2, phase=float(rng.uniform(0, 6.28)))[0], none, none
    if case["eq"] == "burgers":
        return inputs.burgers_modes(int(seed), P, N, x0, x1)[0], none, none
    n_jumps = 8 if bc == "periodic" else 1
    cuts = np.sort(rng.uniform(0.05, 0.95, n_jumps)) if n_jumps > 1 else np.array([0.5])
    rho, u, p = _gas(rng, n_jumps + 1)
    data = inputs.EulerPiecewise(cuts, rho, u, p, gamma=GAMMA, period=(x0, x1) if bc == "periodic" else None)
    n = inputs.n_cells(N, bc, 0)
    q = inputs.euler_taylor(data, inputs.centers(x0, x1, N, n, 0), (x1 - x0) / N, P)
    return q, tuple(q[:, 0, 0]), tuple(q[:, 0, -1])


def _batch_spec(case):
    """Sizes and degrees of the instances: part of the case, not of the data."""
    return inputs.batch_spec(case["B"], case["sizes"], n_lo=case["n_lo"], n_hi=case["n_hi"])


def _batch_states(spec, seed):
    seeds = np.random.default_rng(seed).integers(0, 2 ** 31 - 1, len(spec.N))
    for b in range(len(spec.N)):
        yield _initial_1d(dict(eq="euler", P=int(spec.P[b]), N=int(spec.N[b]), bc="transmissive"), int(seeds[b]))[0]


@functools.lru_cache(maxsize=2)
def _vortex(P, N):
    return inputs.isentropic_vortex(P, N)


def _domain_2d(case):
    if case["eq"] != "euler":
        return (0.0, 2.0, 0.0, 2.0)
    return (-1.0, 1.0, -1.0, 1.0) if case["limiter"] else (-5.0, 5.0, -5.0, 5.0)


def _initial_2d(case, seed):
    """State (nc, ndof, ny, nx) on the original mesh."""
    P, Nx, Ny = case["P"], case["Nx"], case["Ny"]
    x0, x1, y0, y1 = _domain_2d(case)
    rng = np.random.default_rng(seed)
    if case["eq"] != "euler":
        return inputs.taylor2d(inputs.modes2d(int(seed)), P, Nx, Ny)
    if not case["limiter"]:
        # the smooth vortex, somewhere on its periodic square
        return np.roll(_vortex(P, Nx), tuple(int(s) for s in rng.integers(0, Nx, 2)), axis=(2, 3))
    # four quadrant states; the cells a mid line cuts take the mean
    rho, u, p = _gas(rng, 4)
    v = rng.uniform(-0.4, 0.4, 4)
    cons = np.stack([rho, rho * u, rho * v, p / (GAMMA - 1.0) + 0.5 * rho * (u * u + v * v)])
    X, Y = inputs.centers2d(x0, x1, y0, y1, Nx, Ny, 0, case["bc"])
    fx = np.clip(X / ((x1 - x0) / Nx) + 0.5, 0.0, 1.0)      # part of the cell right of x = 0
    fy = np.clip(Y / ((y1 - y0) / Ny) + 0.5, 0.0, 1.0)
    q = np.zeros((4, inputs.ndof2d(P)) + X.shape)
    for c in range(4):
        q[c, 0] = ((1 - fx) * (1 - fy) * cons[c, 0] + fx * (1 - fy) * cons[c, 1]
                   + (1 - fx) * fy * cons[c, 2] + fx * fy * cons[c, 3])
    return q


def prepare(case, seed):
    kind = case["kind"]
    if kind == "batch":
        spec = _batch_spec(case)
        b = binding.Batch("euler", spec.P, spec.N, "transmissive", precision=case["precision"], gamma=GAMMA)
        b.workspace.zero_()                 # the rows' padding is part of what run() returns
        b.rebind()
        for i, q in enumerate(_batch_states(spec, seed)):
            b.write(i, q)
        b.prepare()
        return dict(case=case, batch=b, views=_batch_views(b, spec, case["precision"]))
    if kind in ("run2d", "solve2d"):
        x0, x1, y0, y1 = _domain_2d(case)
        s = binding.Solver2D(case["eq"], case["P"], case["Nx"], case["Ny"], limiter=case["limiter"], bc=case["bc"],
                             x_left=x0, x_right=x1, y_left=y0, y_right=y1, gamma=GAMMA)
    else:
        q, left, right = _initial_1d(case, seed)
        x0, x1 = _domain(case)
        s = binding.Solver(case["eq"], case["P"], case["N"], case["bc"], limiter=case["limiter"],
                           precision=case["precision"], x_left=x0, x_right=x1, gamma=GAMMA, left_state=left,
                           right_state=right)
    if kind in ("run2d", "solve2d"):
        q = _initial_2d(case, seed)
    if kind in ("solve", "solve2d"):
        return dict(case=case, solver=s, q=q)
    s.write(q)
    views = [_views_2d(s, p) if kind == "run2d" else _views_1d(s, p) for p in (0, 1)]
    return dict(case=case, solver=s, views=views, parity=0)


# ---------------------------------------------------------------------------
# One pass.
# ---------------------------------------------------------------------------
def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "batch":
        state["batch"].run(case["steps"], [0.5] + [CFL[p] for p in (1, 2, 3)])
        return state["views"]               # an even number of half-steps: the original meshes
    s, cfl = state["solver"], CFL[case["P"]]
    if kind in ("solve", "solve2d"):
        s.write(state["q"])
        taken = s.advance(case["t_end"], cfl)
        q, info = s.read()
        return [q, info.t, taken]
    if kind == "step":
        s.step(cfl)
        state["parity"] ^= 1
        return state["views"][state["parity"]]
    s.run(case["steps"], cfl)
    return state["views"][0]


# The state where the solver keeps it: the workspace after its control data
# holds point values of both meshes, then derivatives of both meshes, in rows
# padded to 64 cells (include/wcc.h).
def _align(n):
    return (n + 255) // 256 * 256


def _region(ws, offset, nbytes, dtype):
    return ws[offset:offset + nbytes].view(dtype)


def _views_1d(s, parity):
    n, ld = s.ncells(parity), (max(s.ncells(0), s.ncells(1)) + 63) // 64 * 64
    dtype, size = (torch.float64, 8) if s.params.precision == 0 else (torch.float32, 4)
    pb, db = s.nc * ld * 8, s.nc * s.P * ld * size
    p = _region(s.workspace, STATE_OFFSET + parity * _align(pb), pb, torch.float64)
    d = _region(s.workspace, STATE_OFFSET + 2 * _align(pb) + parity * _align(db), db, dtype)
    return [p.view(s.nc, ld)[:, :n], d.view(s.nc, s.P, ld)[:, :, :n]]


def _views_2d(s, parity):
    nc, nd, ny, nx = s.mesh_shape(parity)
    big = max(s.mesh_shape(0)[2] * s.mesh_shape(0)[3], s.Nx * s.Ny)
    plane = (big + 63) // 64 * 64
    qb = nc * nd * plane * 8
    q = _region(s.workspace, STATE_OFFSET + parity * _align(qb), qb, torch.float64)
    return [q.view(nc, nd, plane)[:, :, :nx * ny].unflatten(2, (ny, nx))]


def _batch_rows(spec):
    return [(int(n) + 1 + 63) // 64 * 64 for n in spec.N]


def _batch_views(b, spec, precision):
    """Point values and derivatives of the original meshes, instance after instance (the last pieces of the workspace)."""
    ld = _batch_rows(spec)
    dtype, size = (torch.float64, 8) if precision == "fp64" else (torch.float32, 4)
    pb, db = 3 * sum(ld) * 8, 3 * sum(r * int(p) for r, p in zip(ld, spec.P)) * size
    end = b.workspace.numel()
    return [_region(b.workspace, end - 2 * _align(db) - 2 * _align(pb), pb, torch.float64),
            _region(b.workspace, end - 2 * _align(db), db, dtype)]


# ---------------------------------------------------------------------------
# What one pass cannot do without.  A half-step needs the largest wave speed
# of all cells of the one before, so each is a pass over the state: every old
# cell read and every new cell written once.  States of the small whole
# problems fit one compute unit, so there only the host copy counts.
# ---------------------------------------------------------------------------
_FLOPS_1D = {  # per new cell: limited, unlimited (fused multiply-add = 2)
    "advection": {1: (44, 17), 2: (88, 34), 3: (127, 55), 4: (181, 81)},
    "burgers": {1: (51, 24), 2: (112, 58), 3: (187, 115), 4: (306, 206)},
    "euler": {1: (276, 91), 2: (496, 200), 3: (760, 380), 4: (1158, 664)},
}
_FLOPS_2D = {
    "advection": {1: (110, 50), 2: (300, 120), 3: (560, 240)},
    "burgers": {1: (120, 60), 2: (330, 150), 3: (650, 330)},
    "euler": {1: (800, 350), 2: (2200, 1150), 3: (4300, 2900)},
}


def _half_steps(case):
    """Half-steps of one pass (whole problems: from the end time and a typical wave speed)."""
    if "steps" in case:
        return case["steps"]
    if case["kind"] == "step":
        return 1
    speed = {"advection": 1.0, "burgers": 1.2, "euler": 2.0}[case["eq"]]
    if case["kind"] == "solve2d":
        x0, x1, y0, y1 = _domain_2d(case)
        return max(1, round(case["t_end"] * speed * (case["Nx"] / (x1 - x0) + case["Ny"] / (y1 - y0)) / CFL[case["P"]]))
    x0, x1 = _domain(case)
    return max(1, round(case["t_end"] * speed * case["N"] / (x1 - x0) / CFL[case["P"]]))


def work(case):
    kind = case["kind"]
    k = _half_steps(case)
    if kind == "batch":
        spec, elem = _batch_spec(case), 8 if case["precision"] == "fp64" else 4
        sizes = [(int(n), int(p)) for n, p in zip(spec.N, spec.P)]
        return {"bytes": 2 * k * sum(n * 3 * (8 + p * elem) for n, p in sizes),
                "flops": k * sum(n * _FLOPS_1D["euler"][p][0] for n, p in sizes)}
    column = 0 if case["limiter"] else 1
    if kind in ("run2d", "solve2d"):
        cells, nc = case["Nx"] * case["Ny"], 4 if case["eq"] == "euler" else 1
        per_pass = 2 * cells * nc * inputs.ndof2d(case["P"]) * 8
        flops = cells * _FLOPS_2D[case["eq"]][case["P"]][column]
    else:
        cells, nc = case["N"], 3 if case["eq"] == "euler" else 1
        per_pass = 2 * cells * nc * (8 + case["P"] * (8 if case["precision"] == "fp64" else 4))
        flops = cells * _FLOPS_1D[case["eq"]][case["P"]][column]
    passes = 1 if kind in ("solve", "solve2d") else k
    return {"bytes": passes * per_pass, "flops": k * flops}


# ---------------------------------------------------------------------------
# The half-steps in plain binary64.  Arrays are numpy (small) or torch on the
# GPU (large); only operators and indexing are used on them.
# ---------------------------------------------------------------------------
def _fac(k):
    return float(math.factorial(k))


def _limit_weights(P, st, b):
    """Normalised weights of the candidates with indicators b[0] (high order) and b[1:]."""
    if P == 1:
        w = [(1.0 / (x + EPS)) ** 2 for x in b]
    else:
        r = [st / (x * x + EPS) for x in b]
        w = [1.0 + r[0] * r[0]] + [x * x for x in r[1:]]
    total = sum(w[1:], w[0])
    return [x / total for x in w]


def _limit_1d(P, d, avg, vl, vr):
    """Limited derivatives d[1..P] of one scalar field."""
    s1, s2 = 2.0 * (avg - vl), 2.0 * (vr - avg)
    st = 0.0
    if P == 1:
        b0 = d[1] * d[1]
    else:
        mid = avg - sum(d[k] / (_fac(k + 1) * 2.0 ** k) for k in range(2, P + 1, 2))
        ep = mid + sum(d[k] / (_fac(k) * 2.0 ** k) for k in range(1, P + 1))
        em = mid + sum((-1) ** k * d[k] / (_fac(k) * 2.0 ** k) for k in range(1, P + 1))
        st = ((ep - vr) ** 2 + (em - vl) ** 2) * (d[P] * d[P])
        b0 = 0.0
        for k in range(1, P + 1):           # derivative polynomials squared and integrated over the cell
            c = [d[k + n] / _fac(n) for n in range(P - k + 1)]
            for i in range(len(c)):
                for j in range(len(c)):
                    if (i + j) % 2 == 0:
                        b0 = b0 + c[i] * c[j] / ((i + j + 1) * 2.0 ** (i + j))
    w = _limit_weights(P, st, [b0, s1 * s1, s2 * s2])
    return [None, w[0] * d[1] + w[1] * s1 + w[2] * s2] + [w[0] * d[k] for k in range(2, P + 1)]


def _speed_1d(eq, avg):
    if eq == "advection":
        return abs(avg[0] * 0.0 + 1.0)
    if eq == "burgers":
        return abs(avg[0])
    u = avg[1] / avg[0]
    p = (GAMMA - 1.0) * (avg[2] - 0.5 * avg[1] * u)
    return abs(u) + (GAMMA * p / avg[0]) ** 0.5


def _average_1d(P, q):
    return [x[0] + sum(x[k] / (_fac(k + 1) * 2.0 ** k) for k in range(2, P + 1, 2)) for x in q]


def _half_step_1d(eq, P, limiter, q, lam_old, lam_new, left, right):
    """q[c][k] on the old mesh -> (q, averages) on the new one; lam = dt/dx per old / new cell, left / right the
    parents' indices."""
    nc = len(q)
    T = [[[None] * (P + 1) for _ in range(P + 1)] for _ in range(nc)]      # Taylor coefficients [k][m]
    G = [[[None] * (P + 1) for _ in range(P + 1)] for _ in range(nc)]
    V = [[None] * (P + 1) for _ in range(P + 1)]
    W = [[None] * (P + 1) for _ in range(P + 1)]
    for c in range(nc):
        for k in range(P + 1):
            T[c][k][0] = q[c][k] / _fac(k)

    def mul(X, Y, k, m):
        return sum((X[a][b] * Y[k - a][m - b] for a in range(k + 1) for b in range(m + 1) if a or b),
                   X[0][0] * Y[k][m])

    for m in range(P + 1):
        for k in range(P + 1 - m):
            if eq == "advection":
                G[0][k][m] = T[0][k][m]
            elif eq == "burgers":
                G[0][k][m] = 0.5 * mul(T[0], T[0], k, m)
            else:
                s = sum((-(T[0][a][b] * V[k - a][m - b]) for a in range(k + 1) for b in range(m + 1) if a or b),
                        T[1][k][m])
                V[k][m] = s / T[0][0][0]
                kin = mul(T[1], V, k, m)
                p = (GAMMA - 1.0) * (T[2][k][m] - 0.5 * kin)
                W[k][m] = T[2][k][m] + p
                G[0][k][m], G[1][k][m], G[2][k][m] = T[1][k][m], kin + p, mul(W, V, k, m)
        if m < P:
            for c in range(nc):
                for k in range(P - m):
                    T[c][k][m + 1] = -lam_old * ((k + 1) / (m + 1)) * G[c][k + 1][m]
    flux = [sum(G[c][0][m] / (m + 1) for m in range(P + 1)) for c in range(nc)]
    uR = [q[c][0] + sum(q[c][k] / (_fac(k + 1) * 2.0 ** k) for k in range(1, P + 1)) for c in range(nc)]
    uL = [q[c][0] + sum((-1) ** k * q[c][k] / (_fac(k + 1) * 2.0 ** k) for k in range(1, P + 1)) for c in range(nc)]
    vert = [[_fac(k) * sum(T[c][k][m] for m in range(P + 1 - k)) for k in range(P)] for c in range(nc)]
    avg, d = [], []
    for c in range(nc):
        avg.append(0.5 * (uR[c][left] + uL[c][right]) + lam_new * (flux[c][left] - flux[c][right]))
        x = [None] * (P + 1)
        for k in range(P - 1, -1, -1):
            x[k + 1] = vert[c][k][right] - vert[c][k][left]
            for m in range(3, P - k + 1, 2):
                x[k + 1] = x[k + 1] - 2.0 / (_fac(m) * 2.0 ** m) * x[k + m]
        d.append(x)
    if limiter:
        vl, vr = [vert[c][0][left] for c in range(nc)], [vert[c][0][right] for c in range(nc)]
        if eq != "euler":
            d = [_limit_1d(P, d[0], avg[0], vl[0], vr[0])]
        else:
            rho, u = avg[0], avg[1] / avg[0]
            p = (GAMMA - 1.0) * (avg[2] - 0.5 * avg[1] * u)
            a = (GAMMA * p / rho) ** 0.5
            H = (avg[2] + p) / rho
            b1 = (GAMMA - 1.0) / (a * a)
            b2 = 0.5 * b1 * u * u
            one = rho * 0.0 + 1.0
            L = [[0.5 * (b2 + u / a), -0.5 * (b1 * u + 1.0 / a), 0.5 * b1], [1.0 - b2, b1 * u, -b1],
                 [0.5 * (b2 - u / a), -0.5 * (b1 * u - 1.0 / a), 0.5 * b1]]
            R = [[one, u - a, H - u * a], [one, u, 0.5 * u * u], [one, u + a, H + u * a]]
            out = [[None] + [0.0] * P for _ in range(3)]
            for f in range(3):
                proj = lambda x: L[f][0] * x[0] + L[f][1] * x[1] + L[f][2] * x[2]  # noqa: E731
                cd = [None] + [proj([d[c][k] for c in range(3)]) for k in range(1, P + 1)]
                cd = _limit_1d(P, cd, proj(avg), proj(vl), proj(vr))
                for c in range(3):
                    for k in range(1, P + 1):
                        out[c][k] = out[c][k] + R[f][c] * cd[k]
            d = out
    new = [[avg[c] - sum(d[c][k] / (_fac(k + 1) * 2.0 ** k) for k in range(2, P + 1, 2))] + d[c][1:]
           for c in range(nc)]
    return new, avg


def _parents_1d(N, bc, parity):
    """Indices of the left and right parents of the new cells (Dirichlet: into the old row with both ghosts)."""
    i = np.arange(N)
    if bc == "periodic":
        return (i, (i + 1) % N) if parity == 0 else ((i - 1) % N, i)
    if parity == 0:
        return i, i + 1
    j = np.arange(N + 1)
    if bc == "dirichlet":
        return j, j + 1
    return np.maximum(j - 1, 0), np.minimum(j, N - 1)


def _place(array, device):
    return torch.from_numpy(np.ascontiguousarray(array)).to(device) if device else array


def _device_for(cells):
    return "cuda" if cells > 20000 and torch.cuda.is_available() else None


def _march_1d(case, seed, steps=None, t_end=None):
    """(q as (nc, P+1, n), t, parity) after `steps` half-steps or at t_end."""
    eq, P, N, bc, cfl = case["eq"], case["P"], case["N"], case["bc"], CFL[case["P"]]
    q0, lo, hi = _initial_1d(case, seed)
    if case["precision"] != "fp64":          # the entry point rounds derivatives on write
        q0 = np.concatenate([q0[:, :1], q0[:, 1:].astype(np.float32).astype(np.float64)], axis=1)
    device = _device_for(N)
    q = [[_place(q0[c, k], device) for k in range(P + 1)] for c in range(q0.shape[0])]
    parents = [[_place(x, device) for x in _parents_1d(N, bc, p)] for p in (0, 1)]
    x0, x1 = _domain(case)
    dx, t, parity, done = (x1 - x0) / N, 0.0, 0, 0
    smax = float(_speed_1d(eq, _average_1d(P, q)).max())
    while done < steps if steps is not None else t < t_end:
        dt = cfl * dx / smax
        if t_end is not None and dt >= t_end - t:
            dt = t_end - t
            t = t_end
        else:
            t += dt
        if bc == "dirichlet" and parity == 1:
            cat = torch.cat if device else np.concatenate
            ghost = lambda c, k, s: _place(np.array([s[c] if k == 0 else 0.0]), device)  # noqa: E731
            q = [[cat([ghost(c, k, lo), q[c][k], ghost(c, k, hi)]) for k in range(P + 1)] for c in range(len(q))]
        q, avg = _half_step_1d(eq, P, case["limiter"], q, dt / dx, dt / dx, *parents[parity])
        smax = float(_speed_1d(eq, avg).max())
        parity ^= 1
        done += 1
    stack = torch.stack if device else np.stack
    return stack([stack(x) for x in q]), t, parity


def _march_batch(case, seed):
    """The instances of one degree side by side in one long row, each with its own time step."""
    spec = _batch_spec(case)
    states = list(_batch_states(spec, seed))
    ld, B = _batch_rows(spec), case["B"]
    elem = np.float64 if case["precision"] == "fp64" else np.float32
    p_out, d_out = [None] * B, [None] * B
    for P in (1, 2, 3):
        which = [b for b in range(B) if int(spec.P[b]) == P]
        if not which:
            continue
        device = _device_for(10 ** 9)
        q0 = np.concatenate([states[b] for b in which], axis=2)
        q0[:, 1:] = q0[:, 1:].astype(elem)
        q = [[_place(q0[c, k], device) for k in range(P + 1)] for c in range(3)]
        N = np.array([int(spec.N[b]) for b in which])
        owner, parents = [], []
        for parity in (0, 1):
            n_old, n_new = (N + 1, N) if parity == 0 else (N, N + 1)
            owner.append(_place(np.repeat(np.arange(len(N)), n_old), device))
            start = np.cumsum(n_old) - n_old
            pair = [_parents_1d(int(n), "transmissive", parity) for n in N]
            parents.append([_place(np.concatenate([s + x[side] for s, x in zip(start, pair)]), device)
                            for side in (0, 1)])
        dx = _place(1.0 / N, device)

        def largest(speed, parity):
            if device:
                return torch.zeros(len(N), dtype=torch.float64, device=device).scatter_reduce(
                    0, owner[parity], speed, "amax")
            m = np.zeros(len(N))
            np.maximum.at(m, owner[parity], speed)
            return m

        smax = largest(_speed_1d("euler", _average_1d(P, q)), 0)
        for i in range(case["steps"]):
            lam = CFL[P] * dx / smax / dx
            old, new = i & 1, 1 - (i & 1)
            q, avg = _half_step_1d("euler", P, True, q, lam[owner[old]], lam[owner[new]], *parents[old])
            smax = largest(_speed_1d("euler", avg), new)
        host = np.stack([np.stack([x.cpu().numpy() if device else x for x in row]) for row in q])
        ends = np.cumsum(N + 1)
        for b, n, e in zip(which, N + 1, ends):
            rows = np.zeros((3, P + 1, ld[b]))
            rows[:, :, :n] = host[:, :, e - n:e]
            p_out[b], d_out[b] = rows[:, 0].reshape(-1), rows[:, 1:].reshape(-1)
    return [np.concatenate(p_out), np.concatenate(d_out)]


def _dof(k, l):
    return (k + l) * (k + l + 1) // 2 + l


def _limit_2d(P, D, avg, v):
    """Limited derivatives {(k, l): x} of one field; v: vertex values lower-left, lower-right, upper-right, upper-left."""
    ld, rd, ru, lu = v
    ux = [2 * avg - (ld + lu), rd - ld, rd + ru - 2 * avg, ru - lu]
    uy = [lu - ld, 2 * avg - (ld + rd), ru - rd, lu + ru - 2 * avg]
    beta, st = 0.0, 0.0
    for n in range(1, P + 1):
        for l in range(n + 1):
            k = n - l
            cf = {(e - t, t): D[k + e - t, l + t] / (_fac(e - t) * _fac(t)) for e in range(P - n + 1)
                  for t in range(e + 1)}
            for (s1, t1), x in cf.items():
                for (s2, t2), y in cf.items():
                    a, b = s1 + s2, t1 + t2
                    if a % 2 == 0 and b % 2 == 0:
                        beta = beta + x * y / ((a + 1) * 2.0 ** a * (b + 1) * 2.0 ** b)
    if P >= 2:
        mid = _point_2d(P, avg, D)
        sigma = 0.0
        for (sx, sy), value in zip(((-1, -1), (1, -1), (1, 1), (-1, 1)), v):
            s = mid + sum(sx ** k * sy ** l * x / (2.0 ** (k + l) * _fac(k) * _fac(l)) for (k, l), x in D.items())
            sigma = sigma + (s - value) ** 2
        st = sigma * sum(D[k, P - k] ** 2 for k in range(P + 1))
    w = _limit_weights(P, st, [beta] + [x * x + y * y for x, y in zip(ux, uy)])
    out = {key: w[0] * x for key, x in D.items()}
    for m in range(4):
        out[1, 0] = out[1, 0] + w[m + 1] * ux[m]
        out[0, 1] = out[0, 1] + w[m + 1] * uy[m]
    return out


def _point_2d(P, avg, D):
    return avg - sum(x / (_fac(k + 1) * _fac(l + 1) * 2.0 ** (k + l)) for (k, l), x in D.items()
                     if k % 2 == 0 and l % 2 == 0)


def _rate_2d(eq, avg, dx, dy):
    if eq == "advection":
        return avg[0] * 0.0 + (1.0 / dx + 1.0 / dy)
    if eq == "burgers":
        return abs(avg[0]) * (1.0 / dx + 1.0 / dy)
    u, v = avg[1] / avg[0], avg[2] / avg[0]
    p = (GAMMA - 1.0) * (avg[3] - 0.5 * (avg[1] * u + avg[2] * v))
    c = (GAMMA * p / avg[0]) ** 0.5
    return (abs(u) + c) / dx + (abs(v) + c) / dy


def _half_step_2d(eq, P, limiter, q, dt, dx, dy, lo_x, hi_x, lo_y, hi_y, where):
    """q[c][dof] (rows, columns) on the old mesh -> (q, averages) on the new one."""
    nc = len(q)
    T = [{} for _ in range(nc)]              # Taylor coefficients by (k, l, m)
    F, G = [{} for _ in range(nc)], [{} for _ in range(nc)]
    U, V, W = {}, {}, {}
    for c in range(nc):
        for n in range(P + 1):
            for l in range(n + 1):
                T[c][n - l, l, 0] = q[c][_dof(n - l, l)] / (_fac(n - l) * _fac(l))

    def terms(X, Y, k, l, m):
        return [X[a, b, c] * Y[k - a, l - b, m - c] for a in range(k + 1) for b in range(l + 1)
                for c in range(m + 1) if a or b or c]

    def mul(X, Y, k, l, m):
        return sum(terms(X, Y, k, l, m), X[0, 0, 0] * Y[k, l, m])

    for m in range(P + 1):
        for n in range(P - m + 1):
            for l in range(n + 1):
                k = n - l
                e = (k, l, m)
                if eq == "advection":
                    F[0][e] = G[0][e] = T[0][e]
                elif eq == "burgers":
                    F[0][e] = G[0][e] = 0.5 * mul(T[0], T[0], *e)
                else:
                    U[e] = (T[1][e] - sum(terms(T[0], U, *e), 0.0)) / T[0][0, 0, 0]
                    V[e] = (T[2][e] - sum(terms(T[0], V, *e), 0.0)) / T[0][0, 0, 0]
                    xx, yy, xy = mul(T[1], U, *e), mul(T[2], V, *e), mul(T[1], V, *e)
                    p = (GAMMA - 1.0) * (T[3][e] - 0.5 * (xx + yy))
                    W[e] = T[3][e] + p
                    F[0][e], F[1][e], F[2][e], F[3][e] = T[1][e], xx + p, xy, mul(W, U, *e)
                    G[0][e], G[1][e], G[2][e], G[3][e] = T[2][e], xy, yy + p, mul(W, V, *e)
        for c in range(nc):
            for n in range(P - m):
                for l in range(n + 1):
                    k = n - l
                    T[c][k, l, m + 1] = -(dt / dx * (k + 1) * F[c][k + 1, l, m]
                                          + dt / dy * (l + 1) * G[c][k, l + 1, m]) / (m + 1)

    pick = {"A": (lo_y, lo_x), "B": (hi_y, lo_x), "C": (lo_y, hi_x), "E": (hi_y, hi_x)}

    def at(x, parent):
        rows, cols = pick[parent]
        return x[rows][:, cols]

    def quarter(c, sx, sy):
        return sum(sx ** k * sy ** l * q[c][_dof(k, l)] / (_fac(k + 1) * _fac(l + 1) * 2.0 ** (k + l))
                   for k in range(P + 1) for l in range(P + 1 - k))

    def edge(X, along_y, sign):
        return sum(sign ** s * X[(0, s, m) if along_y else (s, 0, m)] / ((s + 1) * 2.0 ** s * (m + 1))
                   for m in range(P + 1) for s in range(P + 1 - m))

    avg, d, vx = [], [], []
    for c in range(nc):
        h = 0.25 * (at(quarter(c, 1, 1), "A") + at(quarter(c, 1, -1), "B") + at(quarter(c, -1, 1), "C")
                    + at(quarter(c, -1, -1), "E"))
        fu, fd = edge(F[c], True, 1), edge(F[c], True, -1)
        gr, gl = edge(G[c], False, 1), edge(G[c], False, -1)
        fx = (at(fu, "A") - at(fu, "C")) + (at(fd, "B") - at(fd, "E"))
        gy = (at(gr, "A") - at(gr, "B")) + (at(gl, "C") - at(gl, "E"))
        avg.append(h + 0.5 * dt / dx * fx + 0.5 * dt / dy * gy)
        vert = {}
        for n in range(P):
            for l in range(n + 1):
                k = n - l
                x = _fac(k) * _fac(l) * sum(T[c][k, l, m] for m in range(P - n + 1))
                vert[k, l] = {o: at(x, o) for o in "ABCE"}
        vx.append([vert[0, 0][o] for o in "ACEB"])
        D = {}
        for n in range(P, 0, -1):
            for l in range(n + 1):
                k = n - l
                parts = []
                if k >= 1:
                    o = vert[k - 1, l]
                    x = 0.5 * ((o["C"] - o["A"]) + (o["E"] - o["B"]))
                    for s in range(1, P - n + 2, 2):
                        for t in range(0, P - n + 2 - s, 2):
                            if s + t > 1:
                                x = x - 2.0 / (_fac(s) * _fac(t) * 2.0 ** (s + t)) * D[k - 1 + s, l + t]
                    parts.append(x)
                if l >= 1:
                    o = vert[k, l - 1]
                    x = 0.5 * ((o["B"] - o["A"]) + (o["E"] - o["C"]))
                    for t in range(1, P - n + 2, 2):
                        for s in range(0, P - n + 2 - t, 2):
                            if s + t > 1:
                                x = x - 2.0 / (_fac(s) * _fac(t) * 2.0 ** (s + t)) * D[k + s, l - 1 + t]
                    parts.append(x)
                D[k, l] = sum(parts) / len(parts)
        d.append(D)
    if limiter and eq != "euler":
        d = [_limit_2d(P, d[0], avg[0], vx[0])]
    elif limiter:
        gx, gy = d[3][1, 0] / dx, d[3][0, 1] / dy
        g = (gx * gx + gy * gy) ** 0.5
        flat = g == 0.0
        g = where(flat, g + 1.0, g)
        nx, ny = where(flat, g * 0.0 + 1.0, gx / g), where(flat, g * 0.0, gy / g)
        rho, u, v = avg[0], avg[1] / avg[0], avg[2] / avg[0]
        p = (GAMMA - 1.0) * (avg[3] - 0.5 * (avg[1] * u + avg[2] * v))
        a = (GAMMA * p / rho) ** 0.5
        H, un, ut, qq = (avg[3] + p) / rho, u * nx + v * ny, v * nx - u * ny, u * u + v * v
        b1 = (GAMMA - 1.0) / (a * a)
        b2 = 0.5 * qq * b1
        L = [[0.5 * (b2 + un / a), -0.5 * (b1 * u + nx / a), -0.5 * (b1 * v + ny / a), 0.5 * b1],
             [1.0 - b2, b1 * u, b1 * v, -b1], [-ut, -ny, nx, 0.0],
             [0.5 * (b2 - un / a), -0.5 * (b1 * u - nx / a), -0.5 * (b1 * v - ny / a), 0.5 * b1]]
        R = [[1.0, u - a * nx, v - a * ny, H - a * un], [1.0, u, v, 0.5 * qq], [0.0, -ny, nx, ut],
             [1.0, u + a * nx, v + a * ny, H + a * un]]
        out = [{key: 0.0 for key in d[0]} for _ in range(4)]
        for f in range(4):
            proj = lambda x: L[f][0] * x[0] + L[f][1] * x[1] + L[f][2] * x[2] + L[f][3] * x[3]  # noqa: E731
            cd = _limit_2d(P, {key: proj([d[c][key] for c in range(4)]) for key in d[0]}, proj(avg),
                           [proj([vx[c][i] for c in range(4)]) for i in range(4)])
            for c in range(4):
                for key in cd:
                    out[c][key] = out[c][key] + R[f][c] * cd[key]
        d = out
    new = []
    for c in range(nc):
        x = [_point_2d(P, avg[c], d[c])] + [None] * (len(q[c]) - 1)
        for (k, l), value in d[c].items():
            x[_dof(k, l)] = value
        new.append(x)
    return new, avg


def _march_2d(case, seed, steps=None, t_end=None):
    eq, P, bc, cfl = case["eq"], case["P"], case["bc"], CFL[case["P"]]
    Nx, Ny = case["Nx"], case["Ny"]
    x0, x1, y0, y1 = _domain_2d(case)
    dx, dy = (x1 - x0) / Nx, (y1 - y0) / Ny
    q0 = _initial_2d(case, seed)
    device = _device_for(Nx * Ny)
    where = torch.where if device else np.where
    q = [[_place(q0[c, d], device) for d in range(q0.shape[1])] for c in range(q0.shape[0])]
    px = [[_place(x, device) for x in _parents_1d(Nx, bc, p)] for p in (0, 1)]
    py = [[_place(x, device) for x in _parents_1d(Ny, bc, p)] for p in (0, 1)]
    avg = []
    for c in range(len(q)):
        avg.append(q[c][0] + sum(q[c][_dof(k, l)] / (_fac(k + 1) * _fac(l + 1) * 2.0 ** (k + l))
                                 for k in range(0, P + 1, 2) for l in range(0, P + 1 - k, 2) if k + l))
    rate = float(_rate_2d(eq, avg, dx, dy).max())
    t, parity, done = 0.0, 0, 0
    while done < steps if steps is not None else t < t_end:
        dt = cfl / rate
        if t_end is not None and dt >= t_end - t:
            dt = t_end - t
            t = t_end
        else:
            t += dt
        q, avg = _half_step_2d(eq, P, case["limiter"], q, dt, dx, dy, *px[parity], *py[parity], where)
        rate = float(_rate_2d(eq, avg, dx, dy).max())
        parity ^= 1
        done += 1
    stack = torch.stack if device else np.stack
    return stack([stack(x) for x in q]), t, parity


def exact(case, seed):
    """What run() returns on a new state, in binary64 (the number of half-steps of a whole problem has no such value)."""
    kind = case["kind"]
    if kind == "batch":
        return _march_batch(case, seed)
    if kind == "solve":
        q, t, _ = _march_1d(case, seed, t_end=case["t_end"])
        return [q, t, None]
    if kind == "solve2d":
        q, t, _ = _march_2d(case, seed, t_end=case["t_end"])
        return [q, t, None]
    if kind == "run2d":
        return [_march_2d(case, seed, steps=case["steps"])[0]]
    q = _march_1d(case, seed, steps=_half_steps(case))[0]
    return [q[:, 0], q[:, 1:]]

"""Performance cases: what users of the library have it compute.

Each case is one pass through the public entry points of dgweno (DG.run,
Batch.run, run_differentiable) on a state that lives on the GPU.  The problems
and sizes are those of the benchmark and of the paper's experiments, with
ragged meshes, every degree and the Runge-Kutta orders of the convergence
study beside them.  A run continues its state in place, as a simulation does
between two outputs.

exact() evaluates the same scheme with dense float64 matrices in plain torch
(no sum factorisation, no shared faces, gradients by torch.autograd): the
reference that errors are measured against.
"""
import math
import random

import numpy as np
import torch

from paper_2309_12019_amd import dgweno, inputs

ADV, BURGERS, KPP, EULER = inputs.LINADV, inputs.BURGERS, inputs.KPP, inputs.EULER
MODES = {"dg": inputs.MODE_DG, "lo": inputs.MODE_LO, "weno": inputs.MODE_WENO, "zhao": inputs.MODE_ZHAO}
STAGES = {2: 2, 3: 3, 4: 5}  # stages of one step by Runge-Kutta order


# ---------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------
def _run(name, problem, nx, p, steps, ny=1, order=3, mode="weno"):
    c = {"op": "run", "problem": problem, "nx": nx, "ny": ny, "p": p, "mode": mode, "order": order, "steps": steps}
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest configuration: 1D advection of a wave and a pulse, 64 cells; launch latency
        _run("adv1d_64_p2", "adv1d", 64, 2, 100),
        # a row of the convergence study (Table 1: smooth wave, SSP order p + 1, here p = 3 with the five-stage method)
        _run("conv1d_1024_p3_rk4", "conv1d", 1024, 3, 50, order=4),
        # Sod's shock tube at the paper's size (Euler system, reflecting walls)
        _run("sod_128_p2", "sod1d", 128, 2, 100),
        # shock tube on a fine mesh: the Euler system where memory traffic counts
        _run("sod_1m_p2", "sod1d", 1 << 20, 2, 10),
        # solid-body rotation of a hump and a slotted cylinder, the benchmark's mid-size configuration
        _run("rot2d_256_p2", "rot2d", 256, 2, 50, ny=256),
        # the same problem at degree 3 with the fourth-order method that the study pairs it with
        _run("rot2d_256_p3_rk4", "rot2d", 256, 3, 20, ny=256, order=4),
        # degree 4 on a ragged mesh (no multiple of any tile)
        _run("rot2d_701x499_p4", "rot2d", 701, 4, 10, ny=499),
        # the four-quadrant Burgers problem at the paper's size (time-dependent exact exterior state)
        _run("riemann2d_128_p2", "riemann2d", 128, 2, 50, ny=128),
        # the KPP problem at the paper's size (non-convex flux)
        _run("kpp2d_128_p2", "kpp2d", 128, 2, 50, ny=128),
        # the benchmark's headline: 1024^2 P2 Burgers
        _run("burgers2d_1024_p2", "burgers2d", 1024, 2, 20, ny=1024),
        # many independent problems of mixed kind, size and degree in one batch
        {"name": "batch_128_mix", "op": "batch", "mix": 0, "count": 128, "steps": 20},
        # gradient of a functional of the final state with respect to the initial one (forward sweep with
        # checkpoints, then the discrete adjoint)
        {"name": "adjoint_burgers2d_512_p2", "op": "adjoint", "problem": "burgers2d", "nx": 512, "ny": 512, "p": 2,
         "mode": "weno", "order": 3, "steps": 20, "snaps": 8, "keep": False},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng: random.Random):
    kind = rng.choice(["scalar1d", "sod1d", "2d", "2d", "2d", "batch", "adjoint"])
    mode = rng.choice(["weno", "weno", "weno", "weno", "lo", "dg", "zhao"])
    p = rng.randint(1, 4)
    if kind == "batch":
        return {"op": "batch", "mix": rng.randint(1, 10 ** 6), "count": _log(rng, 8, 96), "steps": rng.randint(2, 12)}
    if kind == "adjoint":
        # (Burgers: where a state is constant, as around the rotating bodies, the sensor has no derivative)
        p = rng.randint(1, 3)
        problem = "burgers2d"
        nx = _log(rng, 32, 448)
        steps = rng.randint(4, 16)
        return {"op": "adjoint", "problem": problem, "nx": nx, "ny": max(8, int(nx * rng.uniform(0.5, 1.2))), "p": p,
                "mode": rng.choice(["weno", "weno", "lo"]), "order": 3, "steps": steps,
                "snaps": rng.randint(2, steps), "keep": rng.random() < 0.5}
    order = rng.choice([2, 3, 3, 3, 4])
    if kind == "scalar1d":
        problem, nx, ny = rng.choice(["adv1d", "conv1d", "burgers1d"]), _log(rng, 64, 1 << 20), 1
    elif kind == "sod1d":
        problem, nx, ny = "sod1d", _log(rng, 100, 1 << 20), 1
        mode = "weno" if mode == "dg" else mode  # the tube's jump needs a stabilised scheme
    else:
        problem = rng.choice(["rot2d", "burgers2d", "kpp2d", "riemann2d"])
        nx = _log(rng, 32, 1024)
        if problem == "riemann2d":  # quadrants made of whole cells; the paper's degrees (beyond, its constant states
            nx, p = nx + nx % 2, min(p, 2)  # leave the sensor to rounding)
        ny = nx if problem in ("kpp2d", "riemann2d") else max(8, int(nx * rng.uniform(0.4, 1.1)))
    nl = (p + 1) if ny == 1 else (p + 1) ** 2
    dofs = nx * ny * nl * (3 if problem == "sod1d" else 1)
    if problem == "kpp2d":  # no cheap flux there: fewer steps
        dofs *= 4
    steps = max(1, min(rng.randint(10, 60), int(3e8 / (dofs * STAGES[order]))))
    return _run(None, problem, nx, p, steps, ny=ny, order=order, mode=mode)


# ---------------------------------------------------------------------------
# problems and seeded initial data
# ---------------------------------------------------------------------------
def _workload(problem, nx, ny, p, mode, order, seed):
    rng = np.random.default_rng(seed)
    m = MODES[mode]
    if problem in ("adv1d", "conv1d", "burgers1d"):
        ic = {"adv1d": inputs.sin_plus_pulse, "conv1d": inputs.cos_wave, "burgers1d": inputs.sin_wave}[problem]
        w = inputs.burgers1d(nx, p, mode=m) if problem == "burgers1d" else inputs.adv1d(nx, p, mode=m)
        s = float(rng.uniform())
        w.ic = lambda x: ic((x + s) % 1.0)
    elif problem == "sod1d":
        w = inputs.sod1d(nx, p, mode=m, steps=1)
        # the diaphragm on a cell boundary (a projected jump inside a cell undershoots the low density)
        s, a = 0.5 - round(nx * float(rng.uniform(0.4, 0.6))) / nx, float(rng.uniform(0.9, 1.1))
        w.ic = lambda x: a * inputs.sod_tube(x + s)
    elif problem == "rot2d":
        w = inputs.rot2d(nx, p, seed=seed, mode=m, ny=ny)
    elif problem == "burgers2d":
        w = inputs.burgers2d(nx, p, seed=seed, mode=m, ny=ny, steps=1)
    elif problem == "kpp2d":
        w = inputs.kpp2d(nx, p, mode=m, steps=1)
        s, r = float(rng.uniform(-0.2, 0.2)), float(rng.uniform(-0.2, 0.2))
        w.ic = lambda x, y: inputs.kpp_disc(x + s, y + r)
    else:
        w = inputs.burgers2d_riemann(nx, p, mode=m, steps=1)
        a = float(rng.uniform(-0.1, 0.1))
        w.ic = lambda x, y: inputs.riemann_quadrants(x, y) + a * (torch.sin(math.pi * x) * torch.sin(math.pi * y)) ** 2
    w.rk_order = order
    return w


def _case_workload(c, seed):
    return _workload(c["problem"], c["nx"], c["ny"], c["p"], c["mode"], c["order"], seed)


def _batch_workloads(c, seed):
    """The mix fixes kinds, sizes and degrees; the seed the data."""
    out = []
    for i, w in enumerate(inputs.batch_mix(seed=c["mix"], count=c["count"], steps=c["steps"])):
        problem = "rot2d" if w.dim == 2 else ("adv1d" if w.flux == ADV else "burgers1d")
        out.append(_workload(problem, w.nx, w.ny, w.p, "weno", 3, seed * 1009 + i))
    return out


def _device():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _tensor(a):
    return torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float64, device=_device())


def _legendre(n, x, d=0):
    """d-th derivatives of P_0..P_{n-1} at x: [len(x), n]."""
    cols = []
    for a in range(n):
        e = np.zeros(a + 1)
        e[a] = 1.0
        cols.append(np.polynomial.legendre.legval(x, np.polynomial.legendre.legder(e, d) if d else e))
    return np.stack([np.broadcast_to(v, np.shape(x)) for v in cols], -1)


def _centres(w):
    x = w.x0 + (torch.arange(w.nx, dtype=torch.float64, device=_device()) + 0.5) * w.h
    y = w.y0 + (torch.arange(w.ny, dtype=torch.float64, device=_device()) + 0.5) * w.h
    return x, y


def _initial(w):
    """L2 projection of the initial data with p + 2 Gauss points per axis: [cells, coefficients]."""
    n, q = w.p + 1, w.p + 2
    xi, wt = np.polynomial.legendre.leggauss(q)
    proj = _tensor((_legendre(n, xi) * wt[:, None]) * (np.arange(n) + 0.5))  # [q, n]
    x, y = _centres(w)
    X = x[:, None] + 0.5 * w.h * _tensor(xi)
    if w.dim == 1:
        v = w.ic(X)
        if w.flux == EULER:  # [cells, 3, q] -> component-major coefficients
            return (v.reshape(-1, q) @ proj).reshape(w.nx, 3 * n).contiguous()
        return (v @ proj).contiguous()
    Y = y[:, None] + 0.5 * w.h * _tensor(xi)
    out = torch.empty(w.ny, w.nx, n, n, dtype=torch.float64, device=_device())
    rows = max(1, (1 << 22) // (w.nx * q * q))
    for j in range(0, w.ny, rows):  # a band of rows at a time
        b = Y[j:j + rows]
        shape = (b.shape[0], q, w.nx, q)
        v = w.ic(X[None, None].expand(shape), b[:, :, None, None].expand(shape))
        v = (v.reshape(-1, q) @ proj).reshape(b.shape[0], q, w.nx, n)           # over x
        v = v.permute(0, 2, 3, 1).reshape(-1, q) @ proj                          # over y: [.., a, b]
        out[j:j + rows] = v.reshape(b.shape[0], w.nx, n, n).transpose(2, 3)      # [.., b, a]
    return out.reshape(w.ny * w.nx, n * n).contiguous()


# ---------------------------------------------------------------------------
# a pass through the library
# ---------------------------------------------------------------------------
def prepare(case, seed):
    if case["op"] == "batch":
        ws = _batch_workloads(case, seed)
        b = dgweno.Batch.from_workloads(ws)
        arena = b.empty()
        for view, w in zip(b.views(arena), ws):
            view.copy_(_initial(w))
        return {"op": "batch", "b": b, "U0": arena, "U": b.empty(), "dt": [w.dt() for w in ws], "steps": case["steps"]}
    w = _case_workload(case, seed)
    s = {"op": case["op"], "g": dgweno.DG.from_workload(w), "U0": _initial(w), "dt": w.dt(), "steps": case["steps"]}
    if case["op"] == "run":
        s["U"] = s["g"].empty()
    else:
        s["U0"].requires_grad_(True)
        s["weight"] = _weight(s["U0"], seed)
        s["snaps"], s["keep"] = case["snaps"], case["keep"]
    return s


def _weight(U, seed):
    """The functional's gradient with respect to the final state: weights of a linear observation."""
    g = torch.Generator().manual_seed(int(seed))
    a = torch.rand(2, generator=g, dtype=torch.float64).tolist()
    i = torch.arange(U.numel(), dtype=torch.float64, device=U.device).reshape(U.shape)
    return 1.0 + 0.5 * torch.cos(0.37 * i + 6.0 * a[0]) * (0.5 + a[1])


def run(state):
    if state["op"] == "batch":
        return state["b"].run(state["U"].copy_(state["U0"]), state["dt"], state["steps"])
    if state["op"] == "run":
        state["g"].set_time(0.0)
        return state["g"].run(state["U"].copy_(state["U0"]), state["dt"], state["steps"])
    final = dgweno.run_differentiable(state["g"], state["U0"], state["dt"], state["steps"], state["snaps"],
                                      keep_stages=state["keep"])
    (grad,) = torch.autograd.grad(final, state["U0"], state["weight"])
    return {"final": final.detach(), "grad": grad}


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------
def _operator_flops(dim, p, flux, mode):
    """Arithmetic of one operator evaluation per cell: sum-factorised volume integral, each face once, the
    reconstruction (neighbours' continuations, semi-norms, weights) where the mode has one, dissipation, mass
    inverse and Runge-Kutta combination."""
    n = p + 1
    q = n if flux == ADV else n + 1 if flux in (KPP, EULER) else -(-(3 * p + dim - 1) // 2)
    if dim == 1:
        comps = 3 if flux == EULER else 1
        node = {ADV: 1, BURGERS: 3, EULER: 20}[flux]
        f = comps * (4 * q * n + 8 * n) + q * node + 6 * node
        shift = n * n
    else:
        node = {ADV: 2, BURGERS: 3, KPP: 40}[flux]
        f = 2 * (n * n * q + n * q * q) + node * q * q + 4 * (n * q * q + n * n * q)
        f += 2 * (4 * n * n + 6 * n * q + q * (8 if flux != KPP else 90)) + 4 * n * n + 8 * n * n
        shift = n * n * (n + 1)
    if mode in ("weno", "zhao"):
        nl = n ** dim
        f += 2 * dim * (shift + 5 * nl + 10) + 6 * nl + 30
    return f


def _work(w, mode, steps):
    cells = w.nx * w.ny
    # the five-stage method needs the operator at its third stage state twice only if it is not kept: counted once
    return 2 * 8 * w.ndof, cells * steps * STAGES[w.rk_order] * _operator_flops(w.dim, w.p, w.flux, mode)


def work(case):
    if case["op"] == "batch":
        parts = [_work(w, "weno", case["steps"]) for w in _batch_workloads(case, 0)]
        return {"bytes": sum(b for b, _ in parts), "flops": sum(f for _, f in parts)}
    b, f = _work(_case_workload(case, 0), case["mode"], case["steps"])
    if case["op"] == "adjoint":  # initial state and weights in, final state and gradient out; the reverse of an
        return {"bytes": 2 * b, "flops": 3 * f}  # operator costs about twice the operator
    return {"bytes": b, "flops": f}


def tolerance(case):
    """About four times the largest deviation from exact() over the listed cases and a hundred drawn ones.  Rounding alone
    moves a state by 1e-16 to 3e-15 of its norm; where a state is nearly constant the sensor is a quotient of
    semi-norms at rounding level, which from degree 3 on (their higher derivatives weigh up to 1e5) shows in single
    cells, and so does its derivative in the gradients."""
    p, grad = case.get("p", 4), case["op"] == "adjoint"
    if case["op"] == "batch":
        return {"rel": 1e-11, "max": 2e-8}
    if p <= 2:
        return {"rel": 1e-9, "max": 1e-7} if grad else {"rel": 2e-14, "max": 5e-13}
    if p == 3:
        return {"rel": 1e-8, "max": 1e-6} if grad else {"rel": 2e-12, "max": 1e-9}
    return {"rel": 2e-8, "max": 2e-6}


# ---------------------------------------------------------------------------
# the scheme in plain torch, float64, dense matrices
# ---------------------------------------------------------------------------
def _riemann_exterior(x, y, t):
    """Entropy solution of the four-quadrant Burgers problem: on each line x - y = c the problem is one-dimensional
    with flux u^2 in xi = x + y, and u = (xi - s) / (2 t) with s the minimiser of the Lax-Oleinik functional."""
    if t <= 0.0:
        return inputs.riemann_quadrants(x, y)
    xi, c = x + y, x - y
    a, b = 1.0 - c.abs(), 1.0 + c.abs()
    ul, ur = torch.full_like(xi, 0.5), torch.full_like(xi, -1.0)
    um = torch.where(c > 0, torch.full_like(xi, 0.8), torch.full_like(xi, -0.2))

    def total(s):
        return torch.where(s < a, ul * (s - a), torch.where(s <= b, um * (s - a), um * (b - a) + ur * (s - b)))

    best = val = None
    for s, u, ok in ((a, None, torch.ones_like(a, dtype=torch.bool)), (b, None, torch.ones_like(a, dtype=torch.bool)),
                     (xi - 2 * t * ul, ul, xi - 2 * t * ul <= a),
                     (xi - 2 * t * um, um, (xi - 2 * t * um >= a) & (xi - 2 * t * um <= b)),
                     (xi - 2 * t * ur, ur, xi - 2 * t * ur >= b)):
        f = torch.where(ok, total(s) + (xi - s) ** 2 / (4 * t), torch.full_like(xi, math.inf))
        u = (xi - s) / (2 * t) if u is None else u
        best, val = (u, f) if best is None else (torch.where(f < val, u, best), torch.minimum(f, val))
    return best


class _Scheme:
    """The semi-discrete operator and its steps for one workload; states are [ny, nx, comps, coefficients]."""

    def __init__(self, w, mode):
        self.w, self.mode = w, mode
        p, d = w.p, w.dim
        n = p + 1
        self.n, self.d, self.comps = n, d, 3 if w.flux == EULER else 1
        q = n if w.flux == ADV else n + 1 if w.flux in (KPP, EULER) else -(-(3 * p + d - 1) // 2)
        xi, wt = np.polynomial.legendre.leggauss(q)
        ex, ew = np.polynomial.legendre.leggauss(n)
        one = np.ones((1, 1))

        def tensor(fy, fx):  # y slow, x fast; in 1D the x factor alone
            return np.kron(fy, fx) if d == 2 else fx

        L, D = _legendre(n, xi), _legendre(n, xi, 1)
        lo, hi = _legendre(n, np.array([-1.0])), _legendre(n, np.array([1.0]))
        W = np.kron(wt, wt) if d == 2 else wt
        mass = 1.0 / (np.arange(n) + 0.5)
        M = np.kron(mass, mass) if d == 2 else mass
        self.scale = 2.0 / w.h
        self.V = _tensor(tensor(L, L))
        self.G = [_tensor(tensor(L, D) * W[:, None])] + ([_tensor(tensor(D, L) * W[:, None])] if d == 2 else [])
        fw = wt if d == 2 else np.ones(1)
        self.fw = _tensor(fw)
        one = L if d == 2 else np.ones((1, 1))
        self.face = [[_tensor(tensor(one, lo)), _tensor(tensor(one, hi))]]
        if d == 2:
            self.face.append([_tensor(np.kron(lo, L)), _tensor(np.kron(hi, L))])
        self.minv = _tensor(1.0 / M)
        E, DE = _legendre(n, ex), _legendre(n, ex, 1)
        S = (DE * ew[:, None]).T @ DE
        self.K = _tensor(np.kron(np.diag(mass), S) + np.kron(S, np.diag(mass)) if d == 2 else S)
        # a neighbour's polynomial continued into the cell, projected with the exact rule
        def cont(s):
            return (E * ew[:, None] / 1.0).T @ _legendre(n, ex - 2.0 * s) / mass[:, None]
        I = np.eye(n)
        self.cont = [[_tensor(tensor(I, cont(s))) for s in (-1, 1)]]
        if d == 2:
            self.cont.append([_tensor(np.kron(cont(s), I)) for s in (-1, 1)])
        # the sensor's semi-norm: h^{2k-d} int |D^k v|^2 over 1 <= |k| <= p, on the reference cell
        self.norm = []
        EW = np.kron(ew, ew) if d == 2 else ew
        for k in range(1, p + 1):
            for kx in range(k, -1 if d == 2 else k - 1, -1):
                B = tensor(_legendre(n, ex, k - kx), _legendre(n, ex, kx)) * np.sqrt(EW * 4.0 ** k / 2.0 ** d)[:, None]
                self.norm.append(_tensor(B))
        self.norm = torch.cat(self.norm)
        x, y = _centres(w)
        self.xi = _tensor(xi)
        self.xn = x[:, None] + 0.5 * w.h * self.xi   # [nx, q]
        self.yn = y[:, None] + 0.5 * w.h * self.xi   # [ny, q]
        self.x, self.y, self.q = x, y, q

    def velocity(self, axis, x, y):
        w = self.w
        return w.vx - w.omega * (y - w.cy) if axis == 0 else w.vy + w.omega * (x - w.cx)

    def flux(self, u, axis, v):
        w = self.w
        if w.flux == EULER:
            rho, m, e = u.unbind(2)
            pr = 0.4 * (e - 0.5 * m * m / rho)
            return torch.stack([m, m * m / rho + pr, (e + pr) * m / rho], 2)
        if w.flux == KPP:
            return torch.sin(u) if axis == 0 else torch.cos(u)
        return v * u if w.flux == ADV else 0.5 * v * u * u

    def speed(self, u, axis, v):
        w = self.w
        if w.flux == EULER:
            rho, m, e = u.unbind(2)
            return ((m / rho).abs() + torch.sqrt(1.4 * 0.4 * (e - 0.5 * m * m / rho) / rho))[:, :, None]
        if w.flux == KPP:
            return (torch.cos(u) if axis == 0 else torch.sin(u)).abs()
        return (v + 0.0 * u).abs() if w.flux == ADV else (v * u).abs()

    def neighbour(self, U, axis, s):
        """The neighbour's state on side s, and where there is one ([ny, nx, 1, 1])."""
        ax = 1 - axis
        nb = torch.roll(U, -s, ax)
        has = torch.ones(U.shape[0], U.shape[1], 1, 1, dtype=torch.bool, device=U.device)
        if not (self.w.periodic_x if axis == 0 else self.w.periodic_y):
            edge = (-1 if s > 0 else 0)
            if axis == 0:
                has[:, edge] = False
            else:
                has[edge] = False
        return nb, has

    def sides(self):
        return [(axis, s) for axis in range(self.d) for s in (-1, 1)]

    def seminorm2(self, C):
        v = C @ self.norm.T
        return (v * v).sum(-1, keepdim=True)

    def gamma(self, U):
        w, U = self.w, U[:, :, :1]
        if self.mode in ("dg", "lo"):
            return torch.full_like(U[..., :1], 1.0 if self.mode == "lo" else 0.0)
        cand, has = [U], [torch.ones_like(U[..., :1], dtype=torch.bool)]
        for axis, s in self.sides():
            nb, there = self.neighbour(U, axis, s)
            cand.append(torch.cat([U[..., :1], (nb @ self.cont[axis][(s + 1) // 2].T)[..., 1:]], -1))
            has.append(there)
        m = sum(h.to(U.dtype) for h in has[1:])
        lin = [1.0 - m * w.w_nb] + [torch.full_like(m, w.w_nb)] * (len(cand) - 1)
        beta = [self.seminorm2(c) for c in cand]
        alpha = [torch.where(h, l / (w.eps + b) ** w.r, torch.zeros_like(b)) for h, l, b in zip(has, lin, beta)]
        total = sum(alpha)
        omega = [a / total for a in alpha]
        if self.mode == "zhao":
            dev = sum(torch.where(h, (o / l - 1.0).abs() ** w.theta, torch.zeros_like(o))
                      for h, o, l in zip(has, omega, lin))
            low = torch.minimum(lin[0], torch.where(m > 0, torch.full_like(m, w.w_nb), lin[0]))
            den = (1.0 / low - 1.0).abs() ** w.theta + m
            return torch.where(m > 0, dev / torch.where(m > 0, den, torch.ones_like(den)), torch.zeros_like(dev))
        num2 = self.seminorm2(U - sum(o * c for o, c in zip(omega, cand)))
        den2 = beta[0]
        fine = (num2 > 0) & (den2 > 0)
        ratio = torch.sqrt(torch.where(fine, num2, 0.0 * num2 + 1.0) / torch.where(fine, den2, 0.0 * den2 + 1.0))
        ratio = torch.where(fine, ratio, torch.where(num2 > 0, torch.full_like(ratio, math.inf), 0.0 * ratio))
        g = torch.clamp(ratio, max=1.0) ** w.q
        return torch.where(ratio >= w.b, g, torch.zeros_like(g))

    def rhs(self, U, t):
        w, q = self.w, self.q
        u = U @ self.V.T
        if self.d == 2:
            X = self.xn[None, :, None, None, :].expand(w.ny, w.nx, 1, q, q).reshape(w.ny, w.nx, 1, q * q)
            Y = self.yn[:, None, None, :, None].expand(w.ny, w.nx, 1, q, q).reshape(w.ny, w.nx, 1, q * q)
        else:
            X, Y = self.xn[None, :, None, :], 0.0
        vol = [self.velocity(a, X, Y) for a in range(self.d)]
        R = sum(self.flux(u, a, vol[a]) @ self.G[a] for a in range(self.d))
        # lambda_e: the largest ||F'(u_h)|| at the volume nodes
        if w.lambda_override > 0:
            lam = torch.full_like(U[:, :, :1, :1], w.lambda_override)
        elif w.flux == KPP:
            lam = torch.ones_like(U[:, :, :1, :1])
        elif w.flux == ADV:
            v = vol[0].abs() if self.d == 1 and torch.is_tensor(vol[0]) else None
            lam = (torch.full_like(U[:, :, :1, :1], abs(w.vx)) if self.d == 1 else
                   torch.sqrt(vol[0] ** 2 + vol[1] ** 2).amax(-1, keepdim=True) + 0.0 * U[:, :, :1, :1])
        elif w.flux == EULER:
            lam = self.speed(u, 0, None).amax(-1, keepdim=True)
        else:
            lam = math.hypot(w.vx, w.vy if self.d == 2 else 0.0) * u.abs().amax(-1, keepdim=True)
        R = R - (self.gamma(U) * lam / w.p) * (U @ self.K.T)
        for axis, s in self.sides():
            k = (s + 1) // 2
            um = U @ self.face[axis][k].T
            nb, there = self.neighbour(U, axis, s)
            up = nb @ self.face[axis][1 - k].T
            if self.d == 1:
                x, y = w.x0, 0.0
            elif axis == 0:
                x = (self.x + 0.5 * s * w.h)[None, :, None, None]
                y = self.yn[:, None, None, :]
            else:
                x = self.xn[None, :, None, :]
                y = (self.y + 0.5 * s * w.h)[:, None, None, None]
            if w.flux == EULER:
                out = um * _tensor([1.0, -1.0, 1.0])[:, None]
            elif w.bc_kind == inputs.BC_RIEMANN:
                xx, yy = torch.broadcast_tensors(x, y)
                out = _riemann_exterior(xx, yy, t)
            else:
                out = torch.full_like(um, w.bc_value)
            up = torch.where(there, up, out)
            v = self.velocity(axis, x, y)
            top = torch.maximum(self.speed(um, axis, v), self.speed(up, axis, v))
            if w.flux == KPP:
                shift = 0.0 if axis == 0 else 0.5 * math.pi
                peak = (torch.floor((torch.maximum(um, up) - shift) / math.pi)
                        >= torch.ceil((torch.minimum(um, up) - shift) / math.pi))
                top = torch.where(peak, torch.ones_like(top), top)
            H = 0.5 * s * (self.flux(um, axis, v) + self.flux(up, axis, v)) - 0.5 * top * (up - um)
            R = R - (H * self.fw) @ self.face[axis][k]
        return self.scale * self.minv * R

    def step(self, U, dt, t):
        order = self.w.rk_order
        if order == 2:
            V = U + dt * self.rhs(U, t)
            return 0.5 * U + 0.5 * (V + dt * self.rhs(V, t + dt))
        if order == 3:
            V = U + dt * self.rhs(U, t)
            V = 0.75 * U + 0.25 * (V + dt * self.rhs(V, t + dt))
            return U / 3.0 + (2.0 / 3.0) * (V + dt * self.rhs(V, t + 0.5 * dt))
        # the five-stage fourth-order method of Spiteri and Ruuth, Shu-Osher form: {earlier state: (alpha, beta)}
        rows = ({0: (1.0, 0.391752226571890)},
                {0: (0.444370493651235, 0.0), 1: (0.555629506348765, 0.368410593050371)},
                {0: (0.620101851488403, 0.0), 2: (0.379898148511597, 0.251891774271694)},
                {0: (0.178079954393132, 0.0), 3: (0.821920045606868, 0.544974750228521)},
                {2: (0.517231671970585, 0.0), 3: (0.096059710526147, 0.063692468666290),
                 4: (0.386708617503269, 0.226007483236906)})
        states, times, slopes = [U], [t], []
        for row in rows:
            slopes.append(self.rhs(states[-1], times[-1]))
            states.append(sum(a * states[j] + (b * dt) * slopes[j] if b else a * states[j] for j, (a, b) in row.items()))
            times.append(sum(a * times[j] + b * dt for j, (a, b) in row.items()))
        return states[-1]

    def shape(self, U):
        return U.reshape(self.w.ny, self.w.nx, self.comps, -1)


def _advance(w, mode, steps):
    S, U = _Scheme(w, mode), _initial(w)
    V = S.shape(U)
    for k in range(steps):
        V = S.step(V, w.dt(), k * w.dt())
    return V.reshape(U.shape)


def exact(case, seed):
    if case["op"] == "batch":
        if case["count"] * case["steps"] > 4000:
            return None
        return torch.cat([_advance(w, "weno", case["steps"]).reshape(-1) for w in _batch_workloads(case, seed)])
    w = _case_workload(case, seed)
    if case["op"] == "run":
        return _advance(w, case["mode"], case["steps"])
    S, U = _Scheme(w, case["mode"]), _initial(w)
    path = [S.shape(U)]
    for k in range(case["steps"]):
        path.append(S.step(path[-1], w.dt(), k * w.dt()))
    lam = _weight(U, seed).reshape(path[0].shape)
    for V in path[-2::-1]:
        V = V.detach().requires_grad_(True)
        (lam,) = torch.autograd.grad(S.step(V, w.dt(), 0.0), V, lam)
    return {"final": path[-1].reshape(U.shape), "grad": lam.reshape(U.shape)}

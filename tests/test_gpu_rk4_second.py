"""The 2D fourth-order step forms U4 and the partial sum of the last stage from
one evaluation of L(U3), on every kernel of the per-stage path: against the
operator evaluated on its own (dg_rhs) and the combinations written out, in
plain arithmetic (to a few units in the last place of the state: each step has
five combinations of at most five roundings each, 25 x 1.1e-16, and the
operator's own values enter unchanged) and rounded as the kernels round them
(bit for bit)."""
import ctypes
import math
import subprocess

import numpy as np
import pytest
import torch

from paper_2309_12019_amd import inputs

pytestmark = pytest.mark.gpu

A = ((1.0, 0.391752226571890), (0.444370493651235, 0.555629506348765, 0.368410593050371),
     (0.620101851488403, 0.379898148511597, 0.251891774271694),
     (0.178079954393132, 0.821920045606868, 0.544974750228521),
     (0.517231671970585, 0.096059710526147, 0.063692468666290, 0.386708617503269, 0.226007483236906))


@pytest.mark.parametrize("tile", [(8, 8), (16, 16)])
@pytest.mark.parametrize("kind,n,p", [("rot", 30, 1), ("rot", 30, 4), ("burgers", 21, 2), ("burgers", 139, 3),
                                      ("kpp", 20, 2), ("kpp", 20, 3), ("riemann", 22, 2)])
def test_step_equals_its_combinations(kind, n, p, tile):
    from paper_2309_12019_amd import dgweno
    w = {"rot": lambda: inputs.rot2d(n, p, seed=1, ny=n - 3), "burgers": lambda: inputs.burgers2d(n, p, seed=2, ny=n - 2, steps=1),
         "kpp": lambda: inputs.kpp2d(n, p, steps=1), "riemann": lambda: inputs.burgers2d_riemann(n, p, steps=1)}[kind]()
    w.rk_order = 4
    g = dgweno.DG.from_workload(w)
    g.set_tile(*tile)
    U = g.initial_state(w)
    dt = w.dt()
    (b1,) = A[0][1:]
    t1 = b1 * dt
    t2 = A[1][1] * t1 + A[1][2] * dt
    t3 = A[2][1] * t2 + A[2][2] * dt
    t4 = A[3][1] * t3 + A[3][2] * dt

    def rhs(V, t):
        g.set_time(t)
        return g.rhs(V)

    U1 = U + b1 * dt * rhs(U, 0.0)
    U2 = A[1][0] * U + A[1][1] * U1 + A[1][2] * dt * rhs(U1, t1)
    U3 = A[2][0] * U + A[2][1] * U2 + A[2][2] * dt * rhs(U2, t2)
    L3 = rhs(U3, t3)
    U4 = A[3][0] * U + A[3][1] * U3 + A[3][2] * dt * L3
    ref = A[4][0] * U2 + A[4][1] * U3 + A[4][2] * dt * L3 + A[4][3] * U4 + A[4][4] * dt * rhs(U4, t4)
    g.set_time(0.0)
    V = g.step(U.clone(), dt)
    torch.cuda.synchronize()
    # states that differ by rounding pass through the operator four times; at P3 and P4 its sensor amplifies rounding
    # in nearly constant cells (up to 1e5 of one part in 1e16 there, times dt lambda / h <= 0.1)
    bar = 1e-14 if p <= 2 else 1e-11
    assert float((V - ref).abs().max() / ref.abs().max()) <= bar


SRC = """#include <math.h>
/* v = a un + b (u + dt l), rounded as the stage kernels round it; without a un where a is 0 */
void comb(long n, double a, const double *un, double b, const double *u, double dt, const double *l, double *v) {
  for (long i = 0; i < n; ++i) {
    double w = b * fma(dt, l[i], u[i]);
    v[i] = a != 0.0 ? fma(a, un[i], w) : w;
  }
}
"""


@pytest.fixture(scope="module")
def comb(tmp_path_factory):
    d = tmp_path_factory.mktemp("comb")
    (d / "comb.c").write_text(SRC)
    subprocess.run(["gcc", "-O2", "-ffp-contract=off", "-shared", "-fPIC", str(d / "comb.c"), "-o", str(d / "comb.so"),
                    "-lm"], check=True)
    f = ctypes.CDLL(str(d / "comb.so")).comb
    P, D = ctypes.c_void_p, ctypes.c_double
    f.argtypes = [ctypes.c_long, D, P, D, P, D, P, P]

    def run(a, un, b, u, dt, l):
        un, u, l = (np.ascontiguousarray(x.cpu().numpy()) for x in (un, u, l))
        v = np.empty_like(u)
        f(u.size, a, un.ctypes.data, b, u.ctypes.data, dt, l.ctypes.data, v.ctypes.data)
        return torch.from_numpy(v).cuda()
    return run


# the four-wave and the one-wave kernel on 8x8 tiles (on 256 compute units: the limits of roles_tiles_per_cu), KPP
# tiles of 16, 8 and four waves, the exact exterior state on one and on four waves, and 16x16 tiles
@pytest.mark.parametrize("kind,n,p,mode", [("rot", 30, 1, 2), ("rot", 30, 1, 1), ("rot", 150, 1, 2), ("burgers", 21, 2, 2),
                                           ("burgers", 270, 2, 2), ("rot", 40, 2, 0), ("burgers", 139, 3, 2),
                                           ("rot", 200, 3, 3), ("burgers", 200, 3, 2), ("rot", 30, 4, 2), ("rot", 150, 4, 2),
                                           ("burgers", 200, 4, 1), ("kpp", 20, 2, 2), ("kpp", 160, 1, 2), ("kpp", 200, 2, 2),
                                           ("kpp", 140, 3, 2), ("riemann", 22, 2, 2), ("riemann", 200, 2, 2)])
def test_step_bit_for_bit(kind, n, p, mode, comb):
    from paper_2309_12019_amd import dgweno
    w = {"rot": lambda: inputs.rot2d(n, p, seed=1, ny=n - 3, mode=mode),
         "burgers": lambda: inputs.burgers2d(n, p, seed=2, ny=n - 2, steps=1, mode=mode),
         "kpp": lambda: inputs.kpp2d(n, p, steps=1, mode=mode),
         "riemann": lambda: inputs.burgers2d_riemann(n, p, steps=1, mode=mode)}[kind]()
    w.rk_order = 4
    g = dgweno.DG.from_workload(w)
    dt = w.dt()
    (a10, b10), (a20, a21, b21), (a30, a32, b32), (a40, a43, b43), (a52, a53, b53, a54, b54) = A
    U0 = g.initial_state(w)
    for tile in ((8, 8), (16, 16)):
        g.set_tile(*tile)
        U, V = U0, U0.clone()
        for s in range(2):
            t0 = s * dt
            t1 = a10 * t0 + b10 * dt
            t2 = (a20 * t0 + a21 * t1) + b21 * dt
            t3 = (a30 * t0 + a32 * t2) + b32 * dt
            t4 = (a40 * t0 + a43 * t3) + b43 * dt

            def rhs(X, t):
                g.set_time(t)
                return g.rhs(X)

            U1 = comb(0.0, U, a10, U, dt * b10 / a10, rhs(U, t0))
            U2 = comb(a20, U, a21, U1, dt * b21 / a21, rhs(U1, t1))
            U3 = comb(a30, U, a32, U2, dt * b32 / a32, rhs(U2, t2))
            L3 = rhs(U3, t3)
            U4 = comb(a40, U, a43, U3, dt * b43 / a43, L3)
            W = comb(a52, U2, a53, U3, dt * b53 / a53, L3)
            U = comb(1.0, W, a54, U4, dt * b54 / a54, rhs(U4, t4))
            g.set_time(t0)
            g.step(V, dt)
            torch.cuda.synchronize()
            assert torch.equal(U, V), (tile, s)
        assert torch.isfinite(V).all() and math.isfinite(dt)

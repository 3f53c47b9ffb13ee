"""The reversed sensor for the paper's exponents against the general one
(weno_pow one rounding away from 2), and the adjoint with general exponents
against central differences of the run it differentiates."""
import math

import pytest
import torch

from paper_2309_12019_amd import inputs

pytestmark = pytest.mark.gpu


def _make(kind, p):
    return {"adv1d": lambda: inputs.adv1d(50, p), "burgers1d": lambda: inputs.burgers1d(50, p),
            "rot": lambda: inputs.rot2d(18, p, seed=1, ny=17), "burgers": lambda: inputs.burgers2d(18, p, seed=2, ny=17, steps=1)}[kind]()


def _rough(w, g):
    U = g.initial_state(w)
    gen = torch.Generator(device="cuda").manual_seed(5)
    return U + 0.05 * U.abs().max() * torch.randn(U.shape, generator=gen, device="cuda", dtype=torch.float64)


def _gradient(w, U0, lam, fused, steps=3):
    from paper_2309_12019_amd import dgweno
    g = dgweno.DG.from_workload(w)
    g.set_fused(fused)
    U = U0.clone().requires_grad_(True)
    T = dgweno.run_differentiable(g, U, w.dt(), steps, 2, keep_stages=True)
    (grad,) = torch.autograd.grad(T, U, lam)
    torch.cuda.synchronize()
    return grad


@pytest.mark.parametrize("p", [1, 2, 3, 4])
@pytest.mark.parametrize("kind", ["adv1d", "burgers1d", "rot", "burgers"])
def test_special_and_general_exponents(kind, p):
    from paper_2309_12019_amd import dgweno
    w = _make(kind, p)
    g = dgweno.DG.from_workload(w)
    U0 = _rough(w, g)
    gen = torch.Generator(device="cuda").manual_seed(1)
    lam = torch.randn(U0.shape, generator=gen, device="cuda", dtype=torch.float64)
    grads = {}
    for r in (2.0, math.nextafter(2.0, 3.0)):
        w.r = r
        # (shared and separate launches of the two passes: the same kernels' arithmetic)
        grads[r] = _gradient(w, U0, lam, -1)
        assert torch.equal(grads[r], _gradient(w, U0, lam, 0))
    a, b = grads.values()
    # the weights of rough data (semi-norms of 1e-3 to 1e4 of eps = 1e-6) differ by 1e-15 relative, and by a few
    # roundings of the general power; their derivatives likewise, summed over nine sensor reversals
    assert float((a - b).abs().max() / b.abs().max()) <= 1e-11


@pytest.mark.parametrize("q,r", [(1.0, 3.0), (2.0, 2.0), (1.5, 1.5)])
@pytest.mark.parametrize("kind,p", [("adv1d", 4), ("burgers1d", 1), ("rot", 3), ("burgers", 1), ("burgers", 2)])
def test_general_exponents_against_differences(kind, p, q, r):
    from paper_2309_12019_amd import dgweno
    w = _make(kind, p)
    w.q, w.r = q, r
    g = dgweno.DG.from_workload(w)
    U0 = _rough(w, g)
    gen = torch.Generator(device="cuda").manual_seed(1)
    lam = torch.randn(U0.shape, generator=gen, device="cuda", dtype=torch.float64)
    d = torch.randn(U0.shape, generator=gen, device="cuda", dtype=torch.float64)
    grad = float((_gradient(w, U0, lam, -1) * d).sum())

    def diff(h):
        return float((lam * (g.run(U0 + h * d, w.dt(), 3) - g.run(U0 - h * d, w.dt(), 3))).sum()) / (2 * h)

    # central differences at two widths: truncation falls by 100 between them, rounding is 1e-16 / 1e-6 of the state
    best = min(abs(diff(h) - grad) for h in (1e-5, 1e-6, 1e-7))
    assert best <= 1e-6 * max(abs(grad), float(lam.abs().sum()) * 1e-3)

"""Many steps of a 1D problem per launch (dg_run in 1D) against the per-stage
kernels: the same per-cell arithmetic, so the states must agree bit for bit,
on meshes of one workgroup and of several windows, at the edges of both."""
import numpy as np
import pytest
import torch

from paper_2309_12019_amd import inputs

pytestmark = pytest.mark.gpu


def _problem(kind, n, p, order, mode):
    if kind.startswith("sod"):
        w = inputs.sod1d(n, p, mode=mode, steps=1)
        if n < 8:   # (the tube's jump needs cells on both sides)
            w.ic = lambda x: np.stack([1.0 + 0.2 * np.sin(2 * np.pi * x), 0.0 * x, 2.5 + 0.0 * x], axis=-2)
        elif n % 2:   # the jump between two cells
            w.ic = lambda x: inputs.sod_tube(x - 0.5 / n)
        w.periodic_x = kind == "sod_periodic"
    else:
        w = inputs.burgers1d(n, p, mode=mode) if kind == "burgers" else inputs.adv1d(n, p, mode=mode)
        if kind == "inflow":
            w.periodic_x, w.bc_value = False, 0.3
    w.rk_order = order
    return w


# one workgroup: a cell, its wrap onto itself, wave and workgroup edges;
# windows: one cell more than a workgroup, ragged last windows, and a mesh
# with more windows than compute units (short launches)
# (the Euler system: one workgroup to 128 cells, split windows to 20480)
SIZES = [1, 2, 63, 64, 65, 128, 129, 256, 257, 400, 1000, 20481, 70001]


@pytest.mark.parametrize("n", SIZES)
@pytest.mark.parametrize("order", [2, 3, 4])
@pytest.mark.parametrize("kind,p,mode", [("adv", 2, 2), ("inflow", 4, 2), ("burgers", 1, 3), ("burgers", 3, 2),
                                         ("sod", 2, 2), ("sod_periodic", 3, 2), ("sod", 1, 1), ("inflow", 1, 0)])
def test_line_runs_equal_stage_launches(n, order, kind, p, mode):
    from paper_2309_12019_amd import dgweno
    w = _problem(kind, n, p, order, mode)
    g = dgweno.DG.from_workload(w)
    U0 = g.initial_state(w)
    out = []
    for fused in (-1, 0):
        g.set_fused(fused)
        U = U0.clone()
        for steps in (2, 7, 40):   # two launches, an odd count, several launches
            g.run(U, w.dt(), steps)
        torch.cuda.synchronize()
        out.append(U)
    assert torch.isfinite(out[1]).all()
    assert torch.equal(out[0], out[1])


@pytest.mark.parametrize("order", [3, 4])
@pytest.mark.parametrize("kind", ["sod", "sod_periodic"])
def test_odd_runs_of_one_step_per_launch(order, kind):
    """900001 cells of the Euler system at P4: the plan takes one step per launch (on 256 compute units), so three steps
    end in the second array and are copied back."""
    from paper_2309_12019_amd import dgweno
    w = _problem(kind, 900001, 4, order, 2)
    g = dgweno.DG.from_workload(w)
    U0 = g.initial_state(w)
    out = []
    for fused in (-1, 0):
        g.set_fused(fused)
        out.append(g.run(U0.clone(), w.dt(), 3))
    torch.cuda.synchronize()
    assert torch.isfinite(out[1]).all() and not torch.equal(out[1], U0)
    assert torch.equal(out[0], out[1])


@pytest.mark.parametrize("n", [1, 128, 129, 256, 257, 1000])
@pytest.mark.parametrize("mode", [0, 1])
def test_fourth_order_p4_without_a_sensor(n, mode):
    """The one Euler kernel that takes whole cells at every size."""
    from paper_2309_12019_amd import dgweno
    w = _problem("sod", n, 4, 4, mode)
    g = dgweno.DG.from_workload(w)
    U0 = g.initial_state(w)
    out = []
    for fused in (-1, 0):
        g.set_fused(fused)
        out.append(g.run(U0.clone(), w.dt() / 4, 11))
    torch.cuda.synchronize()
    assert torch.isfinite(out[1]).all() and torch.equal(out[0], out[1])

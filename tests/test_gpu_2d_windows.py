"""2D runs of several steps per launch against one step per launch, bit for bit.

lbm_step of a 2D run keeps windows of nodes on chip over several steps; lbm_step_external
takes one step with the kernel that marches through memory.  Both round alike, so the
states are equal, not close: every 2D kernel family and storage precision, periodic boxes
and walls on either axis, on grids that fit into a window on both axes, on one, on none,
one node more or less than a window, with partial windows at the far sides, and call
lengths of one step, of an odd number and beyond what one launch takes."""

import numpy as np
import pytest

from helpers import gpu_config
from paper_2409_03401_amd import inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

P, W = "periodic", "walls"
FLOW = dict(fluid="D2Q9", drho=0.5, g=(0.0, -1e-4, 0.0), sigma=1e-3, nu=(0.1, 0.05))
FAMILIES = {
    "d2q5": {},
    "d2q9": dict(scalar="D2Q9"),
    "d2q5_flow": FLOW,
    "d2q9_flow": dict(FLOW, scalar="D2Q9"),
    "trt": dict(FLOW, collision="TRT", trt_magic=(3.0 / 16.0, 0.25)),
    "mrt": dict(FLOW, collision="MRT", mrt_rates=((1.2, 1.1, 1.3), (1.1, 1.0, 1.2))),
    "mrt_d2q9": dict(FLOW, scalar="D2Q9", collision="MRT", mrt_rates=((1.2, 1.1, 1.3), (1.1, 1.0, 1.2))),
    "variable_density": dict(FLOW, variable_density=True, drho=3.0),
    "general_kappa": dict(FLOW, kappa=((1.0, 0.1, 0.9), (0.95, -0.05, 1.2))),
    "three_compositions": dict(FLOW, c_eq=((0.2, 0.1, 0.15), (0.6, 0.3, 0.35)), M_C=(0.08, 0.1)),
}
PRECS = ("fp64", "fp32", "fp16", "bf16")


def _check(p, prec, steps):
    from paper_2409_03401_amd.lbm import Simulation
    nx, ny = p["nx"], p["ny"]
    y, x = np.mgrid[0:ny, 0:nx]
    rng = np.random.default_rng(nx * 1000 + ny)
    phi0 = 0.5 + 0.4 * np.sin(0.37 * x + 0.21 * y) * np.cos(0.29 * y - 0.11 * x)
    nc = len(p["c_eq"][0])
    mu = rng.normal(0.0, 0.02, (nc, 1, ny, nx))
    sim = Simulation(gpu_config(p, prec), phi0.reshape(1, ny, nx), mu[0], mu[1], mu_x0=tuple(mu[2:]))
    cur = sim.save()
    nxt = torch.empty_like(cur)
    for n in steps:
        sim.step(n)
        for _ in range(n):
            sim.step_external(cur, nxt)
            cur, nxt = nxt, cur
        got = sim.populations()
        sim.restore(cur)
        assert torch.equal(got, sim.populations()), (nx, ny, prec, n)
    assert bool(torch.isfinite(sim.populations()).all())


@pytest.mark.parametrize("prec", PRECS)
@pytest.mark.parametrize("family", sorted(FAMILIES))
def test_families(family, prec):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    p = inputs._base(75, 50, 1, bc=(W, W, P), M_A=(0.1, 0.07), M_B=(0.06, 0.09))
    p.update(FAMILIES[family])
    _check(p, prec, (1, 7, 20))


# whole grid in a window; one axis in it; neither; a window and one node; one row, one column
GRIDS = [(5, 3), (16, 16), (17, 33), (16, 40), (64, 7), (65, 17), (300, 41), (130, 257), (600, 1), (1, 40), (256, 1)]


@pytest.mark.parametrize("bc", [(P, P, P), (P, W, P), (W, P, P), (W, W, P)])
@pytest.mark.parametrize("nx, ny", GRIDS)
@pytest.mark.parametrize("flow", [False, True])
def test_grids_and_walls(nx, ny, bc, flow):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    p = inputs._base(nx, ny, 1, bc=bc)
    if flow:
        p.update(FLOW)
    for prec in ("fp32", "bf16"):
        _check(p, prec, (2, 13, 40))


@pytest.mark.parametrize("n", [600, 1100])
@pytest.mark.parametrize("flow", [False, True])
def test_large_boxes(n, flow):
    """Sizes at which the large windows and more than one of them per compute unit run."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    p = inputs._base(n, n - 37, 1, bc=(P, W, P))
    if flow:
        p.update(FLOW)
    for prec in ("fp64", "fp32", "fp16"):
        _check(p, prec, (9,))

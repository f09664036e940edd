"""The window kernels of every 2D family against one step per launch, bit for bit, with the
window that runs stated: the plan of each call is evaluated on the host (csrc/plan.hpp) and
has to take the small window on one grid and the family's large window on another.  The
grids are ragged, larger than the window and take several launches a call."""

import numpy as np
import pytest

import plan_program as plans
from helpers import gpu_config
from paper_2409_03401_amd import inputs

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not plans.available(), reason="no C++ compiler")]

torch = pytest.importorskip("torch")

P, W = "periodic", "walls"
FLOW = dict(fluid="D2Q9", drho=0.5, g=(0.0, -1e-4, 0.0), sigma=1e-3, nu=(0.1, 0.05))
MODELS = {
    "bgk": ({}, 0),
    "trt": (dict(collision="TRT", trt_magic=(3.0 / 16.0, 0.25)), plans.TRT),
    "mrt": (dict(collision="MRT", mrt_rates=((1.2, 1.1, 1.3), (1.1, 1.0, 1.2))), plans.MRT),
    "vd": (dict(variable_density=True, drho=3.0), plans.VD),
    "vd_trt": (dict(variable_density=True, drho=3.0, collision="TRT", trt_magic=(3.0 / 16.0, 0.25)),
               plans.VD | plans.TRT),
    "kappa": (dict(kappa=((1.0, 0.1, 0.9), (0.95, -0.05, 1.2))), plans.GK),
    "three": (dict(c_eq=((0.2, 0.1, 0.15), (0.6, 0.3, 0.35)), M_C=(0.08, 0.1)), 0),
}
FAMILIES = [(m, scalar, flow) for m in MODELS for scalar in ("D2Q5", "D2Q9") for flow in (False, True)
            if (flow or not m.startswith("vd")) and not (m == "three" and scalar == "D2Q9")]
STEPS = 20


def _large(model, scalar, flow, prec):
    """Threads of the family's large window (csrc/plan.hpp: large_window)."""
    if not flow or prec == "fp64" or (model in ("mrt", "kappa") and scalar == "D2Q9"):
        return 512
    return 1024


# ragged grids: the first on which the plan takes the large window
LARGE = [(300, 257), (130, 97), (200, 131), (517, 300), (600, 41), (350, 200), (1100, 163)]


@pytest.mark.parametrize("prec", sorted(plans.PRECS))
@pytest.mark.parametrize("model, scalar, flow", FAMILIES)
def test_windows(model, scalar, flow, prec):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2409_03401_amd.lbm import Simulation
    kw, coll = MODELS[model]

    def plan_of(nx, ny, wall_x):
        return plans.windows([dict(nx=nx, ny=ny, n=STEPS, prec=prec, qf=9 if flow else 0, qs=int(scalar[3:]),
                                   nc=3 if model == "three" else 2, wall_x=wall_x, coll=coll)])[0]
    large = _large(model, scalar, flow, prec)
    grid = next(g for g in LARGE if plan_of(*g, False)["nt"] == large)
    for nx, ny, bc, nt in ((75, 50, (W, W, P), 256), (*grid, (P, W, P), large)):
        plan = plan_of(nx, ny, bc[0] == W)
        assert plan["nt"] == nt and plan["launches"] >= 2, plan
        p = inputs._base(nx, ny, 1, bc=bc, M_A=(0.1, 0.07), M_B=(0.06, 0.09))
        p.update(FLOW if flow else {}, scalar=scalar)
        p.update(kw if flow else {k: v for k, v in kw.items() if k != "drho"})
        y, x = np.mgrid[0:ny, 0:nx]
        rng = np.random.default_rng(nx + ny)
        phi0 = 0.5 + 0.4 * np.sin(0.37 * x + 0.21 * y) * np.cos(0.29 * y - 0.11 * x)
        mu = rng.normal(0.0, 0.02, (len(p["c_eq"][0]), 1, ny, nx))
        sim = Simulation(gpu_config(p, prec), phi0.reshape(1, ny, nx), mu[0], mu[1], mu_x0=tuple(mu[2:]))
        cur = sim.save()
        nxt = torch.empty_like(cur)
        sim.step(STEPS)
        for _ in range(STEPS):
            sim.step_external(cur, nxt)
            cur, nxt = nxt, cur
        got = sim.populations()
        sim.restore(cur)
        assert torch.equal(got, sim.populations()), (nx, ny, plan)
        assert bool(torch.isfinite(got).all())

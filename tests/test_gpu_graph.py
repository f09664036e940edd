"""lbm_step recorded in a HIP graph: every replay advances the state by the recorded steps,
as the same number of eager steps does, with eager calls of an even number of steps between
the replays."""

import numpy as np
import pytest

from helpers import gpu_config
from paper_2409_03401_amd import inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

P, W = "periodic", "walls"
FLOW2 = dict(fluid="D2Q9", drho=0.5, g=(0.0, -1e-4, 0.0), sigma=1e-3, nu=(0.1, 0.05))
FLOW3 = dict(FLOW2, fluid="D3Q19", g=(0.0, 0.0, -1e-4))
CASES = {
    "2d": dict(size=(40, 30, 1)),
    "2d_wide": dict(size=(700, 523, 1)),
    "2d_flow_walls": dict(size=(75, 50, 1), bc=(W, W, P), **FLOW2),
    "3d_flow_walls": dict(size=(21, 13, 10), scalar="D3Q7", bc=(W, P, W), **FLOW3),
}


@pytest.mark.parametrize("steps", [2, 4, 6, 10, 20])
@pytest.mark.parametrize("case", sorted(CASES))
def test_replays_advance(case, steps):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2409_03401_amd.lbm import Simulation
    kw = dict(CASES[case])
    nx, ny, nz = kw.pop("size")
    p = inputs._base(nx, ny, nz)
    p.update(kw)
    rng = np.random.default_rng(nx + ny + nz)
    phi0 = 0.5 + 0.3 * rng.uniform(-1.0, 1.0, (nz, ny, nx))
    mu = rng.normal(0.0, 0.02, (2, nz, ny, nx))
    sim = Simulation(gpu_config(p, "fp32"), phi0, mu[0], mu[1])
    eager = Simulation(gpu_config(p, "fp32"), phi0, mu[0], mu[1])
    for s in (sim, eager):
        s.step(steps)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        sim.step(steps)
    for between in (0, 2, 8, 0, 6):
        graph.replay()
        eager.step(steps)
        assert torch.equal(sim.populations(), eager.populations()), (case, steps, between)
        for s in (sim, eager):
            s.step(between)
        torch.cuda.synchronize()
        assert torch.equal(sim.populations(), eager.populations()), (case, steps, between)

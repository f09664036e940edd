"""Moments recorded in a HIP graph, replayed between eager calls of an even number of steps,
on states whose earlier calls took an odd number of launches: every replay gives the fields of
the current state, and the steps are those of a run that records nothing."""

import numpy as np
import pytest

from helpers import gpu_config
from paper_2409_03401_amd import inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

FLOW = dict(fluid="D2Q9", drho=0.5, g=(0.0, -1e-4, 0.0), sigma=1e-3, nu=(0.1, 0.05))
NAMES = ("phi", "cA", "muB")


@pytest.mark.parametrize("flow", [False, True])
@pytest.mark.parametrize("size", [(40, 30), (700, 523)])
def test_recorded_moments(size, flow):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2409_03401_amd.lbm import Simulation
    nx, ny = size
    p = inputs._base(nx, ny, 1)
    p.update(FLOW if flow else {})
    rng = np.random.default_rng(nx)
    phi0 = 0.5 + 0.3 * rng.uniform(-1.0, 1.0, (1, ny, nx))
    mu = rng.normal(0.0, 0.02, (2, 1, ny, nx))
    sim, plain = (Simulation(gpu_config(p, "fp32"), phi0, mu[0], mu[1]) for _ in range(2))
    for s in (sim, plain):
        s.step(2)
        s.moments(NAMES)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        fields = sim.moments(NAMES)
    for n in (2, 4, 2, 10, 6):
        for s in (sim, plain):
            s.step(n)
        graph.replay()
        want = plain.moments(NAMES)
        torch.cuda.synchronize()
        for name in NAMES:
            assert torch.equal(fields[name], want[name]), (n, name)
        assert torch.equal(sim.populations(), plain.populations()), n

"""3D runs on the tile shape and the wall treatment chosen for the grid, bit for bit against
64 x 4 tiles and an exchange at the x and y walls after each step.

A call of several steps bounces back at the x and y walls when it pulls and exchanges the
wall populations once, at its end; single-step calls exchange them after each step.  The
LBM_TILE setting takes the general kernel with the given tile.  The update of a node is the
same in every case, so the populations are equal: grids narrower and wider than a tile, of
odd sizes, of whole 128-byte rows that 64 does or does not divide, one node thin, every
storage precision, with and without flow, on the reduced and the paper's scalar lattices."""

import numpy as np
import pytest

from helpers import gpu_config
from paper_2409_03401_amd import inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

P, W = "periodic", "walls"
FLOW = dict(fluid="D3Q19", drho=0.5, g=(1e-5, 2e-5, -1e-4), sigma=1e-3, nu=(0.1, 0.05))
STEPS = 5


def _run(p, prec, chunks):
    from paper_2409_03401_amd.lbm import Simulation
    nx, ny, nz = p["nx"], p["ny"], p["nz"]
    z, y, x = np.mgrid[0:nz, 0:ny, 0:nx]
    rng = np.random.default_rng(nx * 100 + ny * 10 + nz)
    phi0 = 0.5 + 0.4 * np.sin(0.37 * x + 0.21 * y - 0.17 * z) * np.cos(0.29 * y - 0.11 * x + 0.13 * z)
    mu = rng.normal(0.0, 0.02, (2, nz, ny, nx))
    sim = Simulation(gpu_config(p, prec), phi0, mu[0], mu[1])
    for n in chunks:
        sim.step(n)
    return sim.populations()


def _check(p, prec, monkeypatch):
    monkeypatch.delenv("LBM_TILE", raising=False)
    got = _run(p, prec, (STEPS,))
    assert torch.equal(got, _run(p, prec, (1,) * STEPS))
    monkeypatch.setenv("LBM_TILE", "64x4")
    assert torch.equal(got, _run(p, prec, (1,) * STEPS))
    assert bool(torch.isfinite(got).all())


GRIDS = [(100, 75, 10), (64, 9, 30), (96, 20, 12), (33, 9, 7), (130, 6, 5), (16, 16, 16), (5, 4, 3), (1, 8, 9),
         (257, 3, 4), (128, 5, 1)]


@pytest.mark.parametrize("bc", [(P, P, P), (P, P, W), (W, P, P), (P, W, W), (W, W, W)])
@pytest.mark.parametrize("nx, ny, nz", GRIDS)
def test_grids_and_walls(nx, ny, nz, bc, monkeypatch):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    for flow in (False, True):
        p = inputs._base(nx, ny, nz, scalar="D3Q7", bc=bc)
        if flow:
            p.update(FLOW)
        for prec in ("fp32", "bf16"):
            _check(p, prec, monkeypatch)


@pytest.mark.parametrize("scalar", ["D3Q7", "D3Q19"])
@pytest.mark.parametrize("prec", ["fp64", "fp32", "fp16", "bf16"])
@pytest.mark.parametrize("extra", [{}, dict(collision="TRT"), dict(collision="MRT"), dict(variable_density=True),
                                   dict(kappa=((1.0, 0.1, 0.9), (0.95, -0.05, 1.2)))])
def test_families(scalar, prec, extra, monkeypatch):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    p = inputs._base(75, 22, 9, scalar=scalar, bc=(W, W, W))
    p.update(dict(FLOW, **extra))
    _check(p, prec, monkeypatch)


@pytest.mark.parametrize("tile", ["100x2", "70x3", "48x5", "32x8", "20x12", "16x16", "7x30", "1x100"])
def test_tile_shapes(tile, monkeypatch):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    p = inputs._base(93, 34, 12, scalar="D3Q7", bc=(W, P, W))
    p.update(FLOW)
    monkeypatch.setenv("LBM_TILE", tile)
    got = _run(p, "fp32", (STEPS,))
    monkeypatch.setenv("LBM_TILE", "64x4")
    assert torch.equal(got, _run(p, "fp32", (1,) * STEPS))

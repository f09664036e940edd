"""The library's launch plans (csrc/plan.hpp) evaluated on the host: a small C++ program
that prints them, compiled once per session."""

import functools
import os
import shutil
import subprocess
import tempfile

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include "plan.hpp"
#include <cstdio>
using namespace lbm;
int main() {
    long long n, cols, nz;
    PlanInput in{};
    char what;
    int qs, nc, whole, wall_x, keep_copy;
    while (std::scanf(" %c", &what) == 1) {
        if (what == 'f') {  // chunk of the 3D kernels without the stencil
            if (std::scanf("%lld %lld", &cols, &nz) != 2) return 1;
            std::printf("%d\n", flat_chunk(cols, nz, 256));
        } else if (what == 't') {  // does a tile fit
            int w, h;
            if (std::scanf("%d %d", &w, &h) != 2) return 1;
            std::printf("%d\n", int(tile_fits(w, h)));
        } else if (what == 'g') {  // 3D steps of whole rows: the general kernel?
            int nx, prec, qf;
            if (std::scanf("%d %lld %d %d %d", &nx, &n, &prec, &qf, &qs) != 5) return 1;
            std::printf("%d\n", int(general_tiles(nx, n, prec, qf, qs)));
        } else if (what == 'p') {  // 3D calls with x or y walls: pulled?
            int nx, qf, axes;
            if (std::scanf("%d %lld %d %d %d", &nx, &n, &qf, &qs, &axes) != 5) return 1;
            std::printf("%d\n", int(pull_walls(nx, n, qf, qs, axes)));
        } else if (what == 'n') {  // steps of a launch
            if (std::scanf("%lld %lld %lld", &n, &cols, &nz) != 3) return 1;
            std::printf("%lld\n", steps_of_launch(n, cols, nz));
        } else {  // windows of a 2D call
            if (std::scanf("%d %d %d %d %d %d %lf %d %d %d %d %lld", &in.nx, &in.nz, &in.qf, &qs, &nc, &in.prec,
                           &in.copy_bytes, &whole, &wall_x, &in.coll, &keep_copy, &n) != 12) return 1;
            in.nslots = in.qf + (1 + nc) * qs;
            in.whole = whole != 0;
            in.wall_x = wall_x != 0;
            in.keep_copy = keep_copy != 0;
            in.nt[0] = kSmallWindow;
            in.nt[1] = large_window(in.qf, qs, in.prec, in.coll, nc);
            const BlockPlan p = block_plan(in, n);
            std::printf("%d %lld %d %d %d %d %d\n", p.nt, p.launches, p.g.lw, p.g.hx, p.g.hz, p.g.tiles_x, p.g.tiles_z);
        }
    }
}
"""
FIELDS = ("nt", "launches", "lw", "hx", "hz", "tiles_x", "tiles_z")
PRECS = {"fp64": 0, "fp32": 1, "fp16": 2, "bf16": 3}
TRT, VD, GK, MRT = 1, 2, 4, 8


@functools.lru_cache(maxsize=1)
def _build():
    cxx = shutil.which("g++")
    if cxx is None:
        return None, None
    tmp = tempfile.TemporaryDirectory()
    src, exe = os.path.join(tmp.name, "plans.cpp"), os.path.join(tmp.name, "plans")
    with open(src, "w") as f:
        f.write(PROGRAM)
    subprocess.run([cxx, "-std=c++17", "-O1", "-I", os.path.join(ROOT, "paper_2409_03401_amd", "csrc"), src, "-o", exe],
                   check=True)
    return exe, tmp


def available():
    return _build()[0] is not None


def _ask(lines):
    out = subprocess.run([_build()[0]], input="\n".join(lines), check=True, capture_output=True, text=True).stdout
    return [[int(v) for v in line.split()] for line in out.split("\n") if line]


def flat_chunks(grids):
    """Chunk length for every (columns, planes)."""
    return [r[0] for r in _ask([f"f {c} {n}" for c, n in grids])]


def tile_fits(tiles):
    """Whether a 3D work-group can take every (width, height)."""
    return [bool(r[0]) for r in _ask([f"t {w} {h}" for w, h in tiles])]


def general_tiles(boxes):
    """Whether the steps of every (nx, ny, nz, precision, fluid, scalar directions), rows of whole
    lines, go through the general kernel."""
    return [bool(r[0]) for r in _ask([f"g {nx} {nx * ny * nz} {PRECS[prec]} {qf} {qs}"
                                      for nx, ny, nz, prec, qf, qs in boxes])]


def pull_walls(boxes):
    """Whether calls of several steps of every (nx, ny, nz, fluid, scalar directions, axes with
    walls among x and y) bounce back when they pull."""
    return [bool(r[0]) for r in _ask([f"p {nx} {nx * ny * nz} {qf} {qs} {axes}" for nx, ny, nz, qf, qs, axes in boxes])]


def steps_of_launch(launches):
    """Steps of every (steps of the call, launches, index of the launch)."""
    return [r[0] for r in _ask([f"n {n} {m} {i}" for n, m, i in launches])]


def windows(calls):
    """Windows of every call: dicts with nx, ny, qf, qs, nc, prec, wall_x, coll, n, and keep_copy
    for a state of which a graph holds a call."""
    lines = []
    for c in calls:
        prec, nodes = PRECS[c["prec"]], c["nx"] * c["ny"]
        rest = (1 if c["qf"] else 0) + 1 + c["nc"]
        word = {0: 8, 1: 4}.get(prec, 2)
        moving = c["qf"] + (1 + c["nc"]) * c["qs"] - rest

        def slot(b):
            return (nodes * b + 255) // 256 * 256
        copy = moving * slot(word) + rest * slot(max(word, 4))
        whole = int(c["nx"] * word % 128 == 0)
        lines.append(f"w {c['nx']} {c['ny']} {c['qf']} {c['qs']} {c['nc']} {prec} {copy} {whole} "
                     f"{int(c['wall_x'])} {c['coll']} {int(c.get('keep_copy', False))} {c['n']}")
    return [dict(zip(FIELDS, r)) for r in _ask(lines)]

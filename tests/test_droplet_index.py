"""CPU check of the droplet count's index type: over the anchors of the largest closed grids
the loop of a thread visits what a 64-bit index visits, and ends."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include "euler.hpp"
#include <cstdio>
#include <cstdlib>
#include <initializer_list>
// visits of the thread that starts at `first`, or -1 when the loop does not end
template <class U> long long visits(long long nanchors, U first, U step) {
    long long count = 0;
    const U n = U(nanchors);
    for (U t = first; t < n; t += step)
        if (++count > 100000) return -1;
    return count;
}
int main(int argc, char** argv) {
    for (int i = 1; i + 2 < argc; i += 3) {
        lbm::EulerGeom g{};
        g.d = 3;
        g.nanchors = 1;
        for (int a = 0; a < 3; ++a) g.nanchors *= std::atoll(argv[i + a]) + 1;  // walls on every axis
        const long long step = 1024 * 256;  // the largest grid of the kernel
        for (long long first : {0LL, step - 1}) {
            const long long want = first < g.nanchors ? (g.nanchors - first + step - 1) / step : 0;
            const long long got = g.wide(step) ? visits<unsigned long long>(g.nanchors, first, step)
                                               : visits<unsigned>(g.nanchors, unsigned(first), unsigned(step));
            std::printf("%lld %lld %d\n", want, got, int(g.wide(step)));
        }
    }
}
"""


def test_visits(tmp_path):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no C++ compiler")
    (tmp_path / "visits.cpp").write_text(PROGRAM)
    exe = str(tmp_path / "visits")
    subprocess.run([cxx, "-std=c++17", "-I", os.path.join(ROOT, "paper_2409_03401_amd", "csrc"),
                    str(tmp_path / "visits.cpp"), "-o", exe], check=True)
    top = 2**30
    # nodes below 2^30: 4 (n + 1) anchors up to 2^32, just below, and where a step of the loop wraps
    grids = [(1, 1, top - 1), (1, 1, top - 2), (1, 1, top - 65536), (1, 1, top - 65537), (1, 1, top - 65538),
             (1, 2, top // 2 - 1), (1, 32767, 32767), (1000, 1000, 1000), (100, 75, 50), (1, 1, 1)]
    out = subprocess.run([exe] + [str(v) for g in grids for v in g], check=True, capture_output=True,
                         text=True).stdout.split("\n")
    rows = [tuple(int(v) for v in line.split()) for line in out if line]
    assert len(rows) == 2 * len(grids)
    for i, (want, got, wide) in enumerate(rows):
        assert got == want, (grids[i // 2], want, got)
    # ordinary grids keep the short index
    assert not any(wide for _, _, wide in rows[-6:])

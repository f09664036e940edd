"""CPU checks of the launch plans (csrc/plan.hpp)."""

import random

import pytest

import plan_program as plans

pytestmark = pytest.mark.skipif(not plans.available(), reason="no C++ compiler")

MAX_THREADS = 2**32 - 1  # of a launch along one axis of its grid


def _call(nx, ny, n, prec="fp32", qf=0, qs=5, nc=2, wall_x=False, coll=0, keep_copy=False):
    return dict(nx=nx, ny=ny, n=n, prec=prec, qf=qf, qs=qs, nc=nc, wall_x=wall_x, coll=coll, keep_copy=keep_copy)


def test_flat_chunks_fit_a_launch():
    # up to 2^30 - 1 nodes in one column of tiles, and in many columns
    grids = [(1, 2**24 - 1), (1, 2**24), (1, 2**25 - 2), (1, 2**25), (1, 2**30 - 1), (2, 2**24), (64, 2**20 - 1),
             (2**22, 8), (512, 512), (50, 96), (1, 1)]
    for (cols, nz), zc in zip(grids, plans.flat_chunks(grids)):
        assert zc == 0 or cols * -(-nz // zc) * 256 <= MAX_THREADS, (cols, nz, zc)
    # ordinary grids keep their short chunks
    assert plans.flat_chunks([(50, 96), (512, 512)]) == [1, 2]


def test_tiles_that_fit():
    """A tile given in the environment is taken only when its nodes and its ring fit, also
    where the products of its sides pass 2^32."""
    tiles = [(64, 4), (32, 8), (50, 5), (1, 125), (123, 1), (64, 5), (0, 4), (4, -1), (2**30, 4), (4, 2**30),
             (2**31 - 1, 1), (2**16, 2**16), (2**16 + 1, 2**16 - 1)]
    want = [w > 0 and h > 0 and w * h <= 256 and (w + 2) * (h + 2) <= 464 and 2 * (w + 2) + 2 * h <= 256 for w, h in tiles]
    assert plans.tile_fits(tiles) == want


def test_windows_fit_a_launch():
    # long narrow boxes, whose windows hold lanes beyond the box, and boxes of many halos
    calls = [_call(nx, (2**30 - 1) // nx, n, prec, qf, qs, wall_x=wall)
             for nx in (1, 2, 3, 4, 5, 8, 16, 17, 1000, 32767) for n in (1, 5, 100)
             for prec, qf, qs in (("fp32", 0, 5), ("bf16", 9, 5), ("bf16", 0, 9)) for wall in (False, True)]
    for c, p in zip(calls, plans.windows(calls)):
        assert p["nt"] * p["tiles_x"] * p["tiles_z"] <= MAX_THREADS, (c, p)


def test_steps_of_a_launch():
    """The launches share the steps evenly, also of a call so long that steps times launches
    passes 2^63."""
    cases = [(n, m, i) for n in (1, 2, 7, 200, 10**11, 2**62 + 1) for m in (1, 2, 7, n // 128 + 1)
             if m <= n for i in {0, 1, m // 2, m - 1} if i < m]
    for (n, m, i), steps in zip(cases, plans.steps_of_launch(cases)):
        assert n // m <= steps <= -(-n // m), (n, m, i, steps)
    for n, m in ((1, 1), (7, 3), (200, 7), (1000, 1000)):
        assert sum(plans.steps_of_launch([(n, m, i) for i in range(m)])) == n


def test_windows_are_those_of_the_steps_that_run():
    """The halo of a call's windows is the one that its longest launch needs, whatever the
    number of steps, and with a recorded graph an even call takes an even number of launches."""
    rng = random.Random(5)
    calls = [_call(512, 1, 200, "fp64", wall_x=True), _call(17, 33, 9), _call(200, 200, 6, "fp64"), _call(512, 512, 5)]
    for _ in range(300):
        nx, ny = (int(2 ** rng.uniform(0, 11)) for _ in range(2))
        calls.append(_call(nx, ny, int(2 ** rng.uniform(0, 9)), rng.choice(list(plans.PRECS)), rng.choice((0, 9)),
                           rng.choice((5, 9)), wall_x=rng.random() < 0.5, keep_copy=rng.random() < 0.5))
    ran = 0
    for c, p in zip(calls, plans.windows(calls)):
        if not p["nt"]:
            continue
        ran += 1
        k = -(-c["n"] // p["launches"])
        assert k <= 128 and (not c["keep_copy"] or (p["launches"] - c["n"]) % 2 == 0), (c, p)
        halo = 2 * k - 1 if c["qf"] else k - 1
        bw, bh = 1 << p["lw"], p["nt"] >> p["lw"]
        assert p["hx"] == (0 if c["nx"] <= bw else halo), (c, p)
        assert p["hz"] == (0 if c["ny"] <= bh else halo), (c, p)
    assert ran > 200


def test_launches_are_even_for_graphs_only():
    """Two steps of a large box without flow take one launch of windows; two of one step each,
    which move as many bytes as single steps, only where a graph holds a call."""
    for p, launches in zip(plans.windows([_call(1500, 1300, 2, keep_copy=k) for k in (False, True)]), (1, 2)):
        assert p["nt"] == 0 or p["launches"] == launches, p
    assert plans.windows([_call(1500, 1300, 2)])[0]["launches"] == 1


# Calls whose marching kernel and windows differ by 15 % and more: grid, steps, precision, fluid
# and scalar directions, model, what is allowed (steps a launch; 1: the marching kernel too), and
# us measured for that and for a plan that knew nothing of the models' collisions
MEASURED = [
    (512, 512, 10, "fp16", 0, 9, plans.MRT, (1, 2), 87, 139),
    (256, 128, 6, "fp64", 0, 9, plans.MRT, (3,), 21, 38),
    (300, 257, 6, "fp16", 0, 9, plans.TRT, (3,), 19, 30),
    (512, 256, 6, "fp32", 0, 5, plans.GK, (3,), 18, 28),
    (1100, 1063, 10, "fp32", 0, 5, plans.GK, (2,), 146, 217),
    (2048, 2048, 1, "fp32", 9, 5, plans.TRT, (1,), 167, 219),
    (2048, 2048, 1, "fp32", 9, 5, plans.VD | plans.TRT, (1,), 168, 222),
    # windows that a cautious plan would miss
    (1024, 1024, 40, "fp32", 0, 5, 0, (3, 4, 5), 430, 1060),
    (512, 512, 40, "fp32", 9, 5, 0, (2, 3), 357, 600),
    (150, 93, 100, "fp32", 9, 5, 0, (2, 3, 6), 270, 1490),
]


@pytest.mark.parametrize("nx, ny, n, prec, qf, qs, coll, steps, us, us_other", MEASURED)
def test_plans_where_the_kernels_differ(nx, ny, n, prec, qf, qs, coll, steps, us, us_other):
    p = plans.windows([_call(nx, ny, n, prec, qf, qs, coll=coll)])[0]
    taken = -(-n // p["launches"]) if p["nt"] else 1
    assert taken in steps, p
    if n == 1:
        assert p["nt"] == 0, p


def test_general_kernel_on_whole_rows():
    """Boxes whose rows are whole lines, with us a step measured for the general kernel and for
    64 x 4 tiles."""
    measured = [
        ((80, 80, 80, "fp64", 19, 7), 80, 91), ((160, 160, 160, "fp64", 19, 7), 582, 592),
        ((224, 128, 128, "fp64", 19, 7), 537, 505), ((288, 96, 64, "fp64", 19, 7), 268, 247),
        ((112, 112, 112, "fp64", 19, 19), 446, 435), ((224, 128, 128, "fp64", 19, 19), 1185, 1055),
        ((80, 80, 80, "fp64", 19, 19), 178, 192), ((96, 200, 150, "fp64", 19, 19), 832, 916),
        ((96, 96, 96, "fp32", 19, 7), 59, 71), ((160, 96, 80, "fp32", 19, 7), 95, 90),
        ((224, 128, 128, "fp32", 19, 7), 300, 264), ((96, 200, 150, "fp32", 19, 7), 214, 209),
        ((32, 128, 128, "fp32", 19, 19), 79, 89), ((96, 96, 96, "fp32", 19, 19), 150, 143),
        ((160, 160, 160, "fp32", 19, 19), 674, 619), ((224, 128, 128, "fp32", 19, 19), 647, 530),
        ((96, 96, 96, "fp32", 0, 7), 24, 32), ((224, 128, 128, "fp64", 0, 7), 251, 246),
        ((64, 64, 64, "fp32", 19, 7), 2, 1), ((256, 256, 256, "bf16", 19, 7), 2, 1),
    ]
    for (box, general, tiles), chosen in zip(measured, plans.general_tiles([m[0] for m in measured])):
        assert chosen == (general < tiles), box


def test_walls_pulled_or_exchanged():
    """3D boxes with walls and rows of whole lines, with us a step measured both ways."""
    measured = [
        ((128, 128, 128, 19, 7, 2), 170, 193), ((256, 256, 256, 19, 7, 2), 1304, 1152),
        ((288, 96, 64, 19, 7, 2), 152, 164), ((288, 96, 64, 19, 7, 1), 151, 145),
        ((224, 128, 128, 19, 7, 1), 325, 293), ((112, 112, 112, 19, 7, 1), 223, 228),
        ((64, 64, 64, 19, 19, 1), 47, 65), ((128, 64, 32, 19, 19, 2), 62, 104), ((160, 96, 80, 19, 19, 1), 421, 426),
        ((128, 128, 128, 19, 19, 1), 670, 622), ((224, 128, 128, 19, 19, 2), 1205, 1122),
        ((288, 96, 64, 0, 7, 1), 58, 71), ((224, 128, 128, 0, 19, 1), 364, 383),
    ]
    for (box, pulled, exchanged), chosen in zip(measured, plans.pull_walls([m[0] for m in measured])):
        assert chosen == (pulled < exchanged), box

"""The float transpose adds the samples of each ray's crossing of a cell in
closed form.  Parity with the FP64 oracle where that can go wrong: bricks
with one cell or one short of full, rays exactly along cell faces, many and
few samples a crossing, footprints beyond the staged table in rows and in
columns, views whose rays turn around inside a brick, and values that are
not finite.

Tolerance: a corner sum adds at most a few hundred terms of one sign, each
with under ten roundings of 2^-24, so its relative error is below
(sqrt(300) + 10) 2^-24 < 2e-6; one sample lost or counted twice in the few
thousand voxels here would be 1e-5 or more.
"""

import dataclasses
import math

import numpy as np
import pytest

import oracle
from workloads import Geometry

from gpu_util import require_gpu, rel_l2, to_dev, to_np

pytestmark = pytest.mark.gpu

TOL = 2e-6

BASE = Geometry(16, 16, 5, 2.0, 2.0, 2.5, 30, 14, 2.2, 2.2, 300.0, 450.0, 7)
AXES = (0.0, math.pi / 2, math.pi, 3 * math.pi / 2)

CASES = {
    "one_voxel": dataclasses.replace(BASE, nx=1, ny=1, nz=1),
    # nx + 1 cells: one brick exactly, one cell more, two bricks less one
    "cells_16x17": dataclasses.replace(BASE, nx=15, ny=16),
    "cells_31x33": dataclasses.replace(BASE, nx=30, ny=32, nu=60),
    # odd detectors: central rays along cell faces (odd grid) and along cell
    # centres (even grid), parallel to x and y
    "along_faces": dataclasses.replace(BASE, nx=17, ny=17, nz=3, nu=31, nv=9, n_views=4, angles=AXES),
    "along_centres": dataclasses.replace(BASE, nx=18, ny=18, nz=4, nu=31, nv=9, n_views=4, angles=AXES),
    # about 80 samples a crossing, and at most one
    "short_steps": dataclasses.replace(BASE, step=0.025, n_views=3),
    "long_steps": dataclasses.replace(BASE, step=2.9, n_views=23),
    # thin voxels: crossings of z faces within a cell's column
    "flat_voxels": dataclasses.replace(BASE, hz=0.3, nz=40, nv=24, av=1.2),
    # footprints of more pixels than the table: many rows, and one row wider
    # than the table
    "tall_footprint": dataclasses.replace(BASE, nu=40, au=1.5, nv=300, av=0.08, n_views=3),
    "wide_footprint": dataclasses.replace(BASE, nu=1200, au=0.06, nv=5, n_views=3),
    # close source: wide fans, rays of both signs in one brick
    "wide_angle": dataclasses.replace(BASE, nx=40, ny=40, nz=20, nu=64, nv=40, au=4.0, av=4.0,
                                      sad=62.0, sdd=120.0, n_views=16),
    # the views in chunks that end inside and across batches of 64
    "many_views": dataclasses.replace(BASE, n_views=70),
    "shifted": dataclasses.replace(BASE, x_off=41.3, y_off=-17.7, z_off=6.1, u_off=9.0, nu=80,
                                   n_views=11),
}


# Where a cell spans three detector rows or more, the cells go by columns of
# pixels: the same cases with rows of 0.4 of the height.
SPAN = 3.0
for _n in sorted(set(CASES) - {"flat_voxels", "tall_footprint"}):
    _g = CASES[_n]
    CASES["rows_" + _n] = dataclasses.replace(_g, av=0.4 * _g.av, nv=int(2.5 * _g.nv) + 1)
# the source 2 mm outside the grid's corner: rays over 90 degrees apart in a brick
CASES["rows_at_the_source"] = dataclasses.replace(CASES["rows_wide_angle"], sad=60.0, n_views=9,
                                                  angles=tuple(math.pi / 4 + 0.7 * k for k in range(9)))


def _rows(g):
    return g.hz * g.sdd / (g.sad * g.av)


def test_cases_take_both_ways():
    assert all((_rows(g) >= SPAN) == (n.startswith("rows_") or n == "tall_footprint")
               for n, g in CASES.items())
    # a brick that the source is so near to that no axis leads: its rays
    # through two of the corners run along +-x and +-y, or more apart
    g = CASES["rows_at_the_source"]
    th = g.angles[0]
    src = g.sad * np.array([math.sin(th), -math.cos(th)])
    half = 0.5 * (g.nx + 1) * g.hx
    far = []
    for x in (half - 16 * g.hx, half):
        for y in (-half, 16 * g.hy - half):
            far.append(np.array([x, y]) - src)
    ang = [math.atan2(d[1], d[0]) for d in far]
    spread = max(abs((a - b + math.pi) % (2 * math.pi) - math.pi) for a in ang for b in ang)
    assert spread > math.radians(60), spread


@pytest.mark.parametrize("name", sorted(CASES))
def test_transpose_matches_oracle(name):
    require_gpu()
    import paper_1002_3675_amd as cb
    g = CASES[name]
    print("crossings %s" % name, flush=True)
    rng = np.random.default_rng(41)
    y = rng.uniform(0.5, 4.0, g.proj_shape).astype(np.float32).astype(np.float64)
    f = to_np(cb.Plan(g).backproject(to_dev(y)))
    want = oracle.backproject(g, y)
    assert np.count_nonzero(want) > want.size // 4
    assert rel_l2(f, want) <= TOL, rel_l2(f, want)


@pytest.mark.parametrize("name", sorted(CASES))
def test_double_transpose_matches_oracle(name):
    """The same crossings in double.  Sample positions of under 2000 cells err
    by under 2^-42 of a cell, a few roundings each: 1e-11 on the sums."""
    torch = require_gpu()
    import paper_1002_3675_amd as cb
    g = CASES[name]
    print("double crossings %s" % name, flush=True)
    y = np.random.default_rng(43).uniform(0.5, 4.0, g.proj_shape)
    f = to_np(cb.Plan(g).backproject(torch.from_numpy(y).cuda()))
    want = oracle.backproject(g, y)
    assert rel_l2(f, want) <= 1e-11, rel_l2(f, want)


def test_table_geometries_exceed_the_table():
    """The oversize cases really need parts: lower bounds of a full brick's
    footprint, rows and columns."""
    import paper_1002_3675_amd as cb
    cfg = cb.kernel_config()
    for name, axis in (("tall_footprint", "v"), ("wide_footprint", "u")):
        g = CASES[name]
        half = 0.5 * math.hypot(g.nx * g.hx, g.ny * g.hy)
        mag = g.sdd / (g.sad + half)
        cols = math.floor(min(cfg["brick_x"] * g.hx, cfg["brick_y"] * g.hy) * mag / g.au)
        rows = math.floor(cfg["brick_z"] * g.hz * mag / g.av)
        assert (cols if axis == "u" else cols * rows) > cfg["table_pixels"], name


@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
@pytest.mark.parametrize("name", ["cells_31x33", "rows_cells_31x33"])
def test_a_value_that_is_not_finite_stays_on_its_ray(name, bad):
    """Voxels whose weight for that ray is zero in the oracle keep the value
    they have without it."""
    require_gpu()
    import paper_1002_3675_amd as cb
    g = CASES[name]
    rng = np.random.default_rng(42)
    y = rng.uniform(0.5, 4.0, g.proj_shape).astype(np.float32)
    at = (2, 6, 33)
    one = np.zeros(g.proj_shape)
    one[at] = 1.0
    touched = oracle.backproject(g, one) != 0.0
    y0 = y.copy()
    y0[at] = 0.0
    want = oracle.backproject(g, y0.astype(np.float64))
    y[at] = bad
    f = to_np(cb.Plan(g).backproject(to_dev(y)))
    assert touched.any() and not np.isfinite(f[touched]).any()
    assert np.isfinite(f[~touched]).all()
    assert rel_l2(f[~touched], want[~touched]) <= TOL

"""The transpose where the source is so near that each cell takes its own rays
from the ray table, and beside it the bricks that stay with the staged table
although their footprints exceed it: both types, against the FP64 oracle, and
the time that a near source takes.

Tolerances as for the staged crossings: a corner sum adds at most a few
thousand terms of one sign with under ten roundings of 2^-24 each,
(sqrt(2000) + 10) 2^-24 < 4e-6; in double, sample positions of under 2000
cells err by under 2^-42 of a cell, 1e-11 on the sums."""

import math

import numpy as np
import pytest

import oracle
from workloads import Geometry

from gpu_util import require_gpu, rel_l2, to_dev, to_np

pytestmark = pytest.mark.gpu

TOL = 4e-6

NEAR = {
    # beside the grid's corner, for some views, and further off
    "beside": Geometry(40, 40, 20, 2.0, 2.0, 2.5, 64, 40, 4.0, 4.0, 59.0, 120.0, 9,
                       angles=tuple(math.pi / 4 + 0.7 * k for k in range(9))),
    "radii_1.3": Geometry(33, 31, 30, 2.0, 2.0, 2.0, 70, 66, 2.4, 2.4, 60.0, 108.0, 6),
    "tall": Geometry(24, 26, 90, 2.0, 2.0, 2.0, 60, 151, 2.0, 2.0, 60.0, 110.0, 5),
    # three detector rows a cell and more
    "rows": Geometry(30, 34, 12, 2.0, 2.0, 3.0, 60, 121, 3.0, 0.8, 75.0, 140.0, 6),
    "fine_pixels": Geometry(20, 18, 9, 2.0, 2.0, 2.5, 301, 90, 0.4, 0.5, 50.0, 90.0, 3),
    "off_axis": Geometry(20, 21, 10, 2.0, 2.0, 2.5, 51, 30, 4.0, 4.0, 60.0, 120.0, 7, u_off=10.0,
                         x_off=12.0, y_off=-9.0, z_off=5.0),
    "one_plane": Geometry(33, 31, 1, 2.0, 2.0, 8.0, 70, 30, 2.4, 2.4, 60.0, 108.0, 6),
    "one_column": Geometry(1, 1, 60, 2.0, 2.0, 2.0, 5, 120, 3.0, 2.0, 12.0, 30.0, 12),
    # views in chunks; steps of several cells, and of a twentieth
    "many_views": Geometry(12, 12, 12, 2.0, 2.0, 2.0, 24, 24, 3.0, 3.0, 24.0, 48.0, 70),
    "long_steps": Geometry(33, 31, 30, 2.0, 2.0, 2.0, 70, 66, 2.4, 2.4, 60.0, 108.0, 9, step=7.0),
    "short_steps": Geometry(10, 11, 9, 2.0, 2.0, 2.0, 20, 20, 3.0, 3.0, 21.0, 44.0, 3, step=0.1),
}
FAR = {
    # a brick's footprint beyond the table: 90 x 10 pixels in rows by rays,
    # 50 x 16 by columns, and wider than the table and than its columns
    "far_parts": Geometry(34, 33, 6, 2.0, 2.0, 1.9, 240, 20, 0.6, 0.96, 1500.0, 2200.0, 3),
    "far_column_parts": Geometry(34, 33, 6, 2.0, 2.0, 4.0, 140, 120, 1.0, 0.5, 1500.0, 2200.0, 3),
    "far_wide": Geometry(20, 18, 3, 2.0, 2.0, 1.0, 2600, 5, 0.04, 1.0, 1500.0, 2200.0, 2),
    "far_wide_columns": Geometry(20, 18, 3, 2.0, 2.0, 4.0, 1200, 13, 0.1, 1.6, 1500.0, 2200.0, 2),
    # rays' directions in cells spread by uneven voxels
    "uneven_columns": Geometry(12, 90, 8, 8.0, 1.0, 5.0, 80, 60, 2.0, 1.5, 1000.0, 1500.0, 9),
}
CASES = {**NEAR, **FAR}


@pytest.mark.parametrize("name", sorted(CASES))
def test_transpose_matches_oracle(name):
    torch = require_gpu()
    import paper_1002_3675_amd as cb
    g = CASES[name]
    plan = cb.Plan(g)
    y = np.random.default_rng(91).uniform(0.5, 4.0, g.proj_shape).astype(np.float32)
    want = oracle.backproject(g, y.astype(np.float64))
    assert np.count_nonzero(want) > want.size // 8
    print("near cells %s" % name, flush=True)
    f = to_np(plan.backproject(to_dev(y)))
    assert rel_l2(f, want) <= TOL, rel_l2(f, want)
    f = to_np(plan.backproject(torch.from_numpy(y.astype(np.float64)).cuda()))
    assert rel_l2(f, want) <= 1e-11, rel_l2(f, want)


@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
def test_a_value_that_is_not_finite_stays_on_its_ray(bad):
    require_gpu()
    import paper_1002_3675_amd as cb
    g = NEAR["radii_1.3"]
    y = np.random.default_rng(92).uniform(0.5, 4.0, g.proj_shape).astype(np.float32)
    at = (2, 30, 41)
    one = np.zeros(g.proj_shape)
    one[at] = 1.0
    touched = oracle.backproject(g, one) != 0.0
    y[at] = 0.0
    want = oracle.backproject(g, y.astype(np.float64))
    y[at] = bad
    f = to_np(cb.Plan(g).backproject(to_dev(y)))
    assert touched.any() and not np.isfinite(f[touched]).any()
    assert np.isfinite(f[~touched]).all()
    assert rel_l2(f[~touched], want[~touched]) <= TOL


def test_a_near_source_costs_no_more_than_its_rays():
    """1.15 radii from the axis the transpose takes about 6 of the projector's
    times; with a brick's pixels visited for each of its cells it took 190."""
    torch = require_gpu()
    import paper_1002_3675_amd as cb
    g = Geometry(64, 64, 64, 1.0, 1.0, 1.0, 197, 718, 1.5, 0.45, 52.9, 95.2, 5)
    plan = cb.Plan(g)
    f, y = torch.rand(g.vol_shape, device="cuda"), torch.rand(g.proj_shape, device="cuda")

    def ms(call):
        call()
        a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        a.record()
        for _ in range(5):
            call()
        b.record()
        torch.cuda.synchronize()
        return a.elapsed_time(b) / 5

    assert ms(lambda: plan.backproject(y)) <= 25 * ms(lambda: plan.project(f))

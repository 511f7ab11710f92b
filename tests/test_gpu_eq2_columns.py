"""Eq. (2) with one, two, four and six voxels a lane: grids whose planes leave a
remainder, detectors that hold all, some and none of the imager points, and
a value that is not finite beside the detector's used part, against the FP64
oracle.

Tolerance: a view's term has under ten roundings of 2^-24 and the sum over
the views and the result are in double, so 10 * 2^-24 = 6e-7."""

import dataclasses

import numpy as np
import pytest

import oracle
from workloads import Geometry

from gpu_util import require_gpu, rel_l2, to_dev, to_np

pytestmark = pytest.mark.gpu

TOL = 10 * 2.0 ** -24

ONE = Geometry(37, 29, 11, 2.0, 2.0, 2.5, 40, 18, 2.6, 2.6, 300.0, 450.0, 5)
TWO = dataclasses.replace(ONE, nx=70, ny=66, nz=63, hx=1.0, hy=1.0, hz=0.6)
FOUR = dataclasses.replace(ONE, nx=260, ny=158, nz=65, hx=0.4, hy=0.4, hz=0.5, n_views=3)
SIX = dataclasses.replace(ONE, nx=260, ny=400, nz=99, hx=0.4, hy=0.25, hz=0.33, n_views=3)
NARROW = dict(nu=17, nv=7)          # many imager points beyond the detector
SHIFTED = dict(u_off=30.0, v_off=-9.0)


def _waves(g):
    return -(-g.nx // 64) * -(-g.ny // 4) * 4 * g.nz


@pytest.mark.parametrize("det", [{}, NARROW, SHIFTED], ids=["whole", "narrow", "shifted"])
@pytest.mark.parametrize("g,lo,hi", [(ONE, 0, 8192), (TWO, 8192, 49152), (FOUR, 49152, 196608),
                                     (SIX, 196608, 1 << 40)],
                         ids=["one", "two", "four", "six"])
def test_eq2_matches_oracle(g, lo, hi, det):
    require_gpu()
    import paper_1002_3675_amd as cb
    assert lo <= _waves(g) < hi
    g = dataclasses.replace(g, **det)
    rng = np.random.default_rng(61)
    y = rng.uniform(0.5, 4.0, g.proj_shape).astype(np.float32).astype(np.float64)
    f = to_np(cb.Plan(g).backproject_eq2(to_dev(y)))
    want = oracle.eq2_backproject(g, y)
    assert np.count_nonzero(want) > 0
    assert rel_l2(f, want) <= TOL, rel_l2(f, want)


@pytest.mark.parametrize("nv", [(1 << 20) - 1, (1 << 20) + 5])
def test_eq2_with_many_rows(nv):
    """About 2^20 detector rows, the most that the row's bits are read for,
    and a few more.  Rows are 5e-5 mm high: float rounding of the rows'
    residuals is as before, the row coordinate's error of 2^-32 rows is none."""
    require_gpu()
    import paper_1002_3675_amd as cb
    g = dataclasses.replace(TWO, nu=12, au=13.0, nv=nv, av=5.3e-5, n_views=1)
    rng = np.random.default_rng(63)
    y = rng.uniform(0.5, 4.0, g.proj_shape).astype(np.float32)
    f = to_np(cb.Plan(g).backproject_eq2(to_dev(y)))
    want = oracle.eq2_backproject(g, y.astype(np.float64))
    assert np.count_nonzero(want) > want.size // 2
    assert rel_l2(f, want) <= TOL, rel_l2(f, want)


@pytest.mark.parametrize("sad", [300.3, 301.7, 310.1, 333.3, 350.9])
def test_rows_just_below_the_last(sad):
    """A plane of voxels whose imager points lie on the last detector row but
    for rounding, most of them below it.  The taps of such a point end with
    that row: the first rows, of every view but the first what follows it in
    memory, hold infinities, and no voxel's own taps reach them."""
    require_gpu()
    import paper_1002_3675_amd as cb
    nv, hz = 12, 2.0
    av = hz * 1.5
    g = Geometry(17, 17, 5, 2.0, 2.0, hz, 40, nv, 2.6, av, sad, 1.5 * sad, 8, v_off=-3.5 * av)
    # the plane k = 4 at the isocentre's depth: (k - 2) + (nv - 1) / 2 + 3.5
    assert 2 + 0.5 * (nv - 1) + 3.5 == nv - 1
    y = np.random.default_rng(64).uniform(0.5, 4.0, g.proj_shape).astype(np.float32)
    y[:, 0, :] = 0.0
    want = oracle.eq2_backproject(g, y.astype(np.float64))
    one = np.zeros(g.proj_shape)
    one[:, :2, :] = 1.0
    assert not oracle.eq2_backproject(g, one).any()
    y[:, 0, :] = np.inf
    f = to_np(cb.Plan(g).backproject_eq2(to_dev(y)))
    assert np.isfinite(f).all()
    assert rel_l2(f, want) <= TOL, rel_l2(f, want)


def test_a_value_that_is_not_finite_reaches_its_taps_only():
    require_gpu()
    import paper_1002_3675_amd as cb
    g = dataclasses.replace(TWO, **NARROW)
    rng = np.random.default_rng(62)
    y = rng.uniform(0.5, 4.0, g.proj_shape).astype(np.float32)
    at = (1, 0, 16)  # a corner pixel: the taps beyond it are zero
    one = np.zeros(g.proj_shape)
    one[at] = 1.0
    touched = oracle.eq2_backproject(g, one) != 0.0
    y0 = y.copy()
    y0[at] = 0.0
    want = oracle.eq2_backproject(g, y0.astype(np.float64))
    y[at] = np.inf
    f = to_np(cb.Plan(g).backproject_eq2(to_dev(y)))
    assert touched.any() and not np.isfinite(f[touched]).any()
    assert np.isfinite(f[~touched]).all()
    assert rel_l2(f[~touched], want[~touched]) <= TOL

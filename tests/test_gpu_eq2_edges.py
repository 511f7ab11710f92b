"""Eq. (2) operator at the detector's sides: which pixels a voxel reads there.

On small grids the two pixels of a row come as one load of the pair that holds
those on the detector.  An imager point left of the first pixel centre, right of
the last, above or below takes the one or two pixels that are there and zero for
the others, also on detectors of one and two columns or rows.  Pixels outside a
voxel's four must not reach it: infinities elsewhere leave it finite.

Tolerance: per term the interpolation and the weight round a few times to
2^-24, in sums of positive terms: below 8 x 2^-24 = 5e-7."""

import numpy as np
import pytest

import oracle

from gpu_util import require_gpu, rel_l2, to_dev, to_np

pytestmark = pytest.mark.gpu


def _geom(nu, nv):
    import paper_1002_3675_amd as cb
    return cb.Geometry(16, 16, 16, 2.0, 2.0, 2.0, nu, nv, 2.2, 2.2, 300.0, 450.0, 7)


@pytest.mark.parametrize("nu,nv", [(1, 9), (2, 9), (3, 9), (17, 1), (17, 2), (1, 1), (2, 2),
                                   (16, 16), (33, 40)])
def test_detectors_smaller_than_the_shadow(nu, nv):
    require_gpu()
    import paper_1002_3675_amd as cb
    g = _geom(nu, nv)
    y = np.random.default_rng(41).uniform(0.5, 4.0, g.proj_shape).astype(np.float32)
    got = to_np(cb.Plan(g).backproject_eq2(to_dev(y)))
    assert rel_l2(got, oracle.eq2_backproject(g, y)) < 5e-7


@pytest.mark.parametrize("side", ["left", "right", "low", "high"])
def test_infinite_pixels_reach_only_their_voxels(side):
    require_gpu()
    import paper_1002_3675_amd as cb
    g = _geom(12, 12)
    rows = {"left": np.s_[:, :, 0], "right": np.s_[:, :, -1], "low": np.s_[:, 0, :],
            "high": np.s_[:, -1, :]}[side]
    y = np.random.default_rng(43).uniform(0.5, 4.0, g.proj_shape).astype(np.float32)
    marked = np.zeros(g.proj_shape, np.float32)
    marked[rows] = 1.0
    reached = oracle.eq2_backproject(g, marked) != 0.0
    # (a voxel whose point lies on the next pixel's centre reads a zero weight)
    bad = y.copy()
    bad[rows] = np.inf
    plan = cb.Plan(g)
    clean, got = to_np(plan.backproject_eq2(to_dev(y))), to_np(plan.backproject_eq2(to_dev(bad)))
    assert reached.any() and not reached.all()
    assert (got[~reached] == clean[~reached]).all()
    assert not np.isfinite(got[reached]).any()

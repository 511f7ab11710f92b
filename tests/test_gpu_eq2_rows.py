"""Eq. (2) operator: the fraction of a row that a voxel's imager point lies beyond
a pixel row's centre keeps its relative precision however small it is.  The
middle plane lies 1e-8 mm off the mid-plane, the row beyond the middle one is
all that is not zero, so the result is the weights times that fraction.  With
every number of voxels a lane, against the FP64 oracle.

Tolerance: row coordinates near 10 in double are exact to 2^-49, 2e-7 of a
fraction of 1e-8; interpolation and weights add a few 2^-24."""

import numpy as np
import pytest

import oracle
from workloads import Geometry

from gpu_util import require_gpu, rel_l2, to_dev, to_np

pytestmark = pytest.mark.gpu


# wavefronts of single voxels: one, two, four and six voxels a lane
@pytest.mark.parametrize("n,low,high", [((30, 26, 7), 0, 8192), ((128, 100, 61), 8192, 49152),
                                        ((256, 256, 61), 49152, 196608),
                                        ((512, 400, 67), 196608, 1 << 30)])
def test_small_fractions_of_a_row(n, low, high):
    require_gpu()
    import paper_1002_3675_amd as cb
    nx, ny, nz = n
    assert low <= -(-nx // 64) * -(-ny // 4) * 4 * nz < high
    h = 100.0 / nx
    g = Geometry(nx, ny, nz, h, h, h, 41, 21, 8.0, 8.0, 300.0, 450.0, 3, z_off=1e-8)
    r = np.zeros(g.proj_shape, dtype=np.float32)
    r[:, 11] = np.random.default_rng(95).uniform(0.5, 1.0, (g.n_views, g.nu)).astype(np.float32)
    want = oracle.eq2_backproject(g, r.astype(np.float64))[nz // 2]
    assert (want > 0).all()
    print("eq2 rows %s" % (n,), flush=True)
    f = to_np(cb.Plan(g).backproject_eq2(to_dev(r)))[nz // 2]
    assert rel_l2(f, want) <= 2e-6, rel_l2(f, want)

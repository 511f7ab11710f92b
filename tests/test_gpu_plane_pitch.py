"""The projector spaces the planes of its staged boxes by the LDS banks of the
tile's rays: detectors that leave ragged tiles, rays along x, along y and
oblique, pixels finer and coarser than the voxels (few and many cells a
tile), boxes up to the LDS capacity, narrow rows beside wide ones, more
sample pieces than one box table holds, against the FP64 oracle.

Tolerance: the samples' float coordinates err by under 2^-24 of a segment's
extent (at most 128 cells a segment here), so weights err by under 2^-17;
with volume values in [a, 2a] neighbours differ by at most half the smaller
sum of a sample's value, and errors of the 10^2 and more samples of a ray are
independent to first order: 2^-17 / 2 / 10 = 3.8e-7, next to the float
roundings of the lerps and sums, under ten of 2^-24: 6e-7.  Together 1e-6."""

import math

import numpy as np
import pytest

import oracle
from workloads import Geometry

from gpu_util import require_gpu, rel_l2, to_dev, to_np

pytestmark = pytest.mark.gpu

TOL = 1e-6
ANGLES = (0.0, math.pi / 2, math.pi / 4, 2.5)

CASES = {
    "cells-as-pixels": Geometry(48, 44, 40, 2.0, 2.0, 2.0, 45, 35, 3.0, 3.0, 400.0, 600.0, 4,
                                angles=ANGLES),
    "fine-pixels": Geometry(40, 40, 9, 2.0, 2.0, 6.0, 70, 50, 1.2, 1.2, 400.0, 600.0, 4,
                            angles=ANGLES),
    "coarse-pixels": Geometry(60, 60, 33, 1.0, 1.0, 1.0, 23, 17, 2.4, 2.4, 400.0, 600.0, 4,
                              angles=ANGLES),
    "thin-planes": Geometry(36, 40, 70, 2.0, 2.0, 0.7, 33, 31, 3.0, 3.0, 400.0, 600.0, 4,
                            angles=ANGLES),
    "one-tile": Geometry(5, 3, 2, 2.0, 2.0, 2.0, 3, 2, 3.0, 3.0, 400.0, 600.0, 4, angles=ANGLES),
    "long-rays": Geometry(1200, 20, 20, 1.0, 1.0, 1.0, 18, 18, 1.5, 1.5, 1500.0, 2200.0, 2,
                          angles=(math.pi / 2, math.pi / 2 + 0.002)),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_spaced_planes_match_oracle(name):
    require_gpu()
    import paper_1002_3675_amd as cb
    g = CASES[name]
    rng = np.random.default_rng(31)
    f = rng.uniform(0.01, 0.02, g.vol_shape).astype(np.float32).astype(np.float64)
    if name == "long-rays":  # more pieces than one table of boxes
        assert g.nx * g.hx / (0.5 * g.hx) > 128 * cb.kernel_config()["tile_chunk"]
    print("projecting %s" % name, flush=True)
    y = to_np(cb.Plan(g).project(to_dev(f)))
    want = oracle.project(g, f)
    assert np.count_nonzero(want) > want.size // 4
    assert rel_l2(y, want) <= TOL, rel_l2(y, want)

"""The projector with steps of many spacings, given explicitly: a segment's
samples then lie so many rows and planes from its origin that the LDS
addresses of their terms exceed what floats hold exactly.  Against the FP64
oracle.

Tolerance: a coordinate is rounded to 2^-24 of its distance l from the
segment's origin, as is its increment, so a sample's weights err by 2^-23 l
cells and its value by that times the volume's spread, here at most its
values; 4e-6 covers the sums' own roundings."""

import math

import numpy as np
import pytest

import oracle
from workloads import Geometry

from gpu_util import require_gpu, rel_l2, to_dev, to_np

pytestmark = pytest.mark.gpu


def _thin(nz, hz, step, views):
    # planes thin against the step, far off the mid-plane: steep rays
    return Geometry(40, 36, nz, 5.0, 5.0, hz, 40, 60, 4.0, 0.3, 1000.0, 1500.0, views, step=step,
                    v_off=900.0, z_off=600.0)


CASES = {
    "terms_beyond_floats": _thin(1, 0.02, 4.8, 12),
    "terms_at_the_bound": _thin(1, 0.04, 4.8, 12),
    "terms_below": _thin(2, 0.2, 4.8, 12),
    "cubes": Geometry(60, 50, 40, 1.0, 1.0, 1.0, 70, 60, 1.6, 1.6, 300.0, 450.0, 5, step=9.0),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_long_steps_match_oracle(name):
    require_gpu()
    import paper_1002_3675_amd as cb
    g = CASES[name]
    f = np.random.default_rng(83).uniform(0.01, 0.02, g.vol_shape).astype(np.float32)
    want = oracle.project(g, f.astype(np.float64))
    assert np.count_nonzero(want) > 100
    slope = (0.5 * (g.nv - 1) * g.av + g.v_off) / g.sdd
    far = 256 * g.step * max(slope / math.hypot(1.0, slope) / g.hz, 1.0 / g.hx, 1.0 / g.hy)
    print("long steps %s: %.0f cells from an origin" % (name, far), flush=True)
    y = to_np(cb.Plan(g).project(to_dev(f)))
    assert rel_l2(y, want) <= 4e-6 + 2.0 ** -23 * far, rel_l2(y, want)

"""The double projector with one to sixteen lanes to a ray: rays of few and of
many samples, detectors whose width leaves part of a block, fine pixels, and
rays that miss the grid, against the FP64 oracle.

Tolerance: sample positions of under 2000 cells err by under 2^-42 of a cell,
a few roundings each, and the order of a ray's sum moves it by roundings of
2^-53: 1e-11."""

import math

import numpy as np
import pytest

import oracle
from workloads import Geometry

from gpu_util import require_gpu, rel_l2, to_np

pytestmark = pytest.mark.gpu

ANGLES = (0.0, math.pi / 2, math.pi / 4, 2.5)


def _geom(n, nz, nu, nv, pitch=1.8):
    h = 150.0 / n
    return Geometry(n, n - 1, nz, h, h, 1.3 * h, nu, nv, pitch * h, pitch * h, 400.0, 600.0, 4,
                    angles=ANGLES)


# samples a ray on average, from and below; geometry
CASES = {
    "one": (0, 24, _geom(9, 5, 13, 7)),
    "two": (24, 64, _geom(24, 20, 21, 15)),
    "four": (64, 96, _geom(45, 34, 37, 19)),
    "eight": (96, 160, _geom(70, 50, 41, 23)),
    "sixteen": (160, 1000, _geom(129, 70, 35, 17)),
    "one_of_fine_pixels": (64, 1000, _geom(60, 40, 67, 33, 0.7)),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_double_projection_matches_oracle(name):
    torch = require_gpu()
    import paper_1002_3675_amd as cb
    lo, hi, g = CASES[name]
    plan = cb.Plan(g)
    mean = plan.samples / (g.nu * g.nv * g.n_views)
    assert lo <= mean < hi, mean
    assert (g.au * g.sad < 0.5 * g.sdd * min(g.hx, g.hy)) == (name == "one_of_fine_pixels")
    f = np.random.default_rng(71).uniform(0.0, 0.02, g.vol_shape)
    print("double projection, %s" % name, flush=True)
    y = to_np(plan.project(torch.from_numpy(f).cuda()))
    want = oracle.project(g, f)
    assert np.count_nonzero(want) > want.size // 4
    assert rel_l2(y, want) <= 1e-11, rel_l2(y, want)

"""The projector's pieces that exceed the LDS box, staged in halves of the tile:
pixels of about a voxel with planes as thick, thinner and few, ragged
detectors, halves that miss the grid, halves that do not fit either, against
the FP64 oracle.

Tolerance: as for the projector with spaced planes, 1e-6 (coordinates within
2^-24 of a segment, neighbours that differ by at most the smaller value, ten
roundings of the sums)."""

import math

import numpy as np
import pytest

import oracle
from workloads import Geometry

from gpu_util import require_gpu, rel_l2, to_dev, to_np

pytestmark = pytest.mark.gpu

TOL = 1e-6


def _angles(n):
    return tuple(0.1 + 2 * math.pi * k / n for k in range(n))


CASES = {
    # 16 x 16 x 12 tiles and more: at least two a CU
    "cubes": Geometry(96, 90, 88, 1.5, 1.5, 1.5, 99, 93, 2.3, 2.3, 500.0, 750.0, 14),
    "thin_planes": Geometry(80, 84, 120, 1.5, 1.5, 0.75, 90, 101, 2.1, 2.1, 500.0, 750.0, 14),
    "beside_the_grid": Geometry(80, 80, 60, 1.5, 1.5, 1.5, 100, 130, 2.3, 2.3, 500.0, 750.0, 12,
                                angles=_angles(12), u_off=20.0, v_off=40.0),
    "too_large_halves": Geometry(100, 100, 100, 1.0, 1.0, 1.0, 100, 99, 4.5, 3.0, 500.0, 750.0, 14),
    "few_tiles": Geometry(96, 90, 88, 1.5, 1.5, 1.5, 99, 93, 2.3, 2.3, 500.0, 750.0, 4),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_pieces_in_halves_match_oracle(name):
    require_gpu()
    import paper_1002_3675_amd as cb
    g = CASES[name]
    tiles = -(-g.nu // 16) * -(-g.nv // 16) * g.n_views
    assert (tiles >= 512) == (name != "few_tiles"), tiles
    cfg = cb.kernel_config()
    mag = g.sad / g.sdd
    u, step = cfg["tile_u"] * g.au * mag, 0.5 * min(g.hx, g.hy, g.hz)
    side = math.sqrt(0.5) * (u + cfg["tile_chunk"] * step) / g.hx + 3.5
    box = side * side * min(cfg["tile_v"] * g.av * mag / g.hz + 3.5, g.nz + 2)
    assert box > cfg["tile_lds_floats"], box
    f = np.random.default_rng(81).uniform(0.01, 0.02, g.vol_shape).astype(np.float32)
    print("projecting %s" % name, flush=True)
    y = to_np(cb.Plan(g).project(to_dev(f)))
    want = oracle.project(g, f.astype(np.float64))
    assert np.count_nonzero(want) > want.size // 8
    assert rel_l2(y, want) <= TOL, rel_l2(y, want)

"""Projecting in halves of the tile gives the same floats, bit for bit: a scan of
enough tiles for halves against the same views a few at a time, which are too
few.  Pieces whose halves all fit the LDS box, and pieces some of whose halves
exceed it, by a lower bound of the box (no margins, no borders)."""

import dataclasses
import math

import numpy as np
import pytest

from workloads import Geometry

from gpu_util import require_gpu, to_dev

pytestmark = pytest.mark.gpu

CASES = {
    "halves_fit": Geometry(96, 90, 88, 1.5, 1.5, 1.5, 99, 93, 2.3, 2.3, 500.0, 750.0, 14),
    "thin_planes": Geometry(80, 84, 120, 1.5, 1.5, 0.75, 90, 101, 2.1, 2.1, 500.0, 750.0, 14),
    "some_exceed": Geometry(90, 96, 90, 1.0, 1.0, 1.0, 110, 110, 2.46, 1.98, 500.0, 750.0, 15),
}


def _tiles(g):
    return -(-g.nu // 16) * -(-g.nv // 16) * g.n_views


@pytest.mark.parametrize("name", sorted(CASES))
def test_halves_equal_whole_tiles(name):
    torch = require_gpu()
    import paper_1002_3675_amd as cb
    g = CASES[name]
    angles = tuple(0.05 + 2 * math.pi * k / g.n_views for k in range(g.n_views))
    g = dataclasses.replace(g, angles=angles)
    cfg = cb.kernel_config()
    mag = g.sad / g.sdd
    u, l = cfg["tile_u"] * g.au * mag, cfg["tile_chunk"] * 0.5 * min(g.hx, g.hy, g.hz)
    side = math.sqrt(0.5) * (u + l) / g.hx
    half = side * side * 0.5 * cfg["tile_v"] * g.av * mag / g.hz
    assert _tiles(g) >= 512
    assert (half > cfg["tile_lds_floats"]) == (name == "some_exceed"), half
    f = to_dev(np.random.default_rng(84).uniform(0.0, 0.02, g.vol_shape).astype(np.float32))
    print("halves bit for bit %s" % name, flush=True)
    y = cb.Plan(g).project(f)
    for k in range(0, g.n_views, 5):
        part = dataclasses.replace(g, n_views=len(angles[k:k + 5]), angles=angles[k:k + 5])
        assert _tiles(part) < 512
        assert torch.equal(cb.Plan(part).project(f), y[k:k + 5]), k

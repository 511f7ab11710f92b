"""The transpose of scans whose bricks' views are kept for a slab of the views at a
time: by rays and by columns, float and double, with the update, and again on
the same plan, against the FP64 oracle.  Tolerances as for the crossings."""

import dataclasses

import numpy as np
import pytest

import oracle
from workloads import Geometry

from gpu_util import require_gpu, rel_l2, to_dev, to_np

pytestmark = pytest.mark.gpu

# 64 bytes per brick and view are more than 8 GiB; the last slab is shorter
CASES = {
    "rays": Geometry(300, 290, 200, 1.0, 1.0, 1.0, 24, 16, 20.0, 20.0, 1000.0, 1500.0, 1901),
    "columns": Geometry(250, 300, 230, 1.0, 1.0, 1.2, 30, 500, 16.0, 0.55, 1000.0, 1500.0, 1923),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_slabs_match_oracle(name):
    torch = require_gpu()
    import paper_1002_3675_amd as cb
    g = CASES[name]
    bricks = -(-(g.nx + 1) // 16) * -(-(g.ny + 1) // 16) * (g.nz + 1)
    assert 64 * bricks * g.n_views > 8 << 30
    rng = np.random.default_rng(103)
    y = rng.uniform(0.5, 4.0, g.proj_shape).astype(np.float32)
    # (the oracle is slow: every 150th view holds data)
    keep = np.zeros(g.n_views, bool)
    keep[::150] = True
    keep[-1] = True
    y[~keep] = 0.0
    angles = tuple(2 * np.pi * k / g.n_views for k in np.flatnonzero(keep))
    few = dataclasses.replace(g, n_views=len(angles), angles=angles)
    want = oracle.backproject(few, y[keep].astype(np.float64))
    print("slabs %s" % name, flush=True)
    plan = cb.Plan(g)
    f = plan.backproject(to_dev(y))
    assert rel_l2(to_np(f), want) <= 2e-6, rel_l2(to_np(f), want)
    assert torch.equal(plan.backproject(to_dev(y)), f)
    f0 = rng.uniform(0.0, 1.0, g.vol_shape).astype(np.float32)
    got = to_np(plan.backproject_update(to_dev(y), to_dev(f0), 1e-3))
    assert rel_l2(got, f0 - 1e-3 * want) <= 2e-6
    del f
    f = plan.backproject(torch.from_numpy(y.astype(np.float64)).cuda())
    assert rel_l2(to_np(f), want) <= 1e-11, rel_l2(to_np(f), want)

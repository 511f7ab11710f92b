"""The transpose of grids whose views are cut into chunks: counts of views at the
least that a chunk keeps, one less and one more, for bricks few, some and many,
in both types against the FP64 oracle (tolerances as for the crossings)."""

import numpy as np
import pytest

import oracle
from workloads import Geometry

from gpu_util import require_gpu, rel_l2, to_dev, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,views", [(12, 7), (12, 8), (12, 9), (12, 33), (56, 15), (56, 16),
                                     (56, 17), (70, 15), (70, 16), (70, 17), (80, 31), (80, 32), (80, 33)])
def test_chunks_match_oracle(n, views):
    torch = require_gpu()
    import paper_1002_3675_amd as cb
    g = Geometry(n, n, n, 2.0, 2.0, 2.0, n + 5, n // 2, 3.0, 3.0, 700.0, 1050.0, views)
    y = np.random.default_rng(101).uniform(0.5, 4.0, g.proj_shape).astype(np.float32)
    want = oracle.backproject(g, y.astype(np.float64))
    print("chunks %d / %d" % (n, views), flush=True)
    plan = cb.Plan(g)
    f = to_np(plan.backproject(to_dev(y)))
    assert rel_l2(f, want) <= 2e-6, rel_l2(f, want)
    f = to_np(plan.backproject(torch.from_numpy(y.astype(np.float64)).cuda()))
    assert rel_l2(f, want) <= 1e-11, rel_l2(f, want)

"""Several TV steps in one launch: grids that end on, one short of and one
beyond the boxes' strides for one, two and three steps a launch (30 x 14 x 8,
28 x 12 x 8, 26 x 10 x 6 voxels), both step counts a launch is chosen for,
and rows too long for the boxes, against single steps bit for bit and the
FP64 oracle.

Tolerance: a step's update is a few terms of a size below that of z with
about twenty roundings of 2^-24, and the step is a contraction, so k steps
stay below 20 k 2^-24 (k <= 9: 1.1e-5)."""

import numpy as np
import pytest

import oracle

from gpu_util import require_gpu, rel_l2, to_dev, to_np

pytestmark = pytest.mark.gpu

H = np.array([0.9, 1.1, 2.3])


def _case(shape, seed):
    rng = np.random.default_rng(seed)
    return to_dev(rng.uniform(-0.002, 0.02, shape)), to_dev(rng.uniform(0.0, 0.02, shape))


@pytest.mark.parametrize("shape", [(1, 1, 1), (2, 1, 3), (8, 14, 30), (9, 15, 31), (16, 12, 28),
                                   (17, 13, 29), (6, 10, 26), (7, 11, 27), (13, 31, 53),
                                   (96, 126, 131)])
@pytest.mark.parametrize("nonneg", [True, False])
def test_steps_equal_single_steps(shape, nonneg):
    torch = require_gpu()
    import paper_1002_3675_amd as cb
    print("tv steps %s" % (shape,), flush=True)
    g, z0 = _case(shape, 51)
    z, at = z0, 0
    for k in (1, 2, 3, 4, 5, 7, 8, 9):
        while at < k:
            z = cb.tv_prox(g, z, H, 600.0, 1e-3, 1, nonneg=nonneg)
            at += 1
        assert torch.equal(cb.tv_prox(g, z0, H, 600.0, 1e-3, k, nonneg=nonneg), z), k
    if nonneg:
        want = oracle.tv_prox(g.double().cpu().numpy(), z0.double().cpu().numpy(), H, 600.0,
                              1e-3, 9)
        assert rel_l2(to_np(z), want) <= 20 * 9 * 2.0 ** -24


def test_rows_beyond_the_boxes_offsets():
    require_gpu()
    import paper_1002_3675_amd as cb
    shape = (1, 1, 2 ** 24 + 5)
    g, z0 = _case(shape, 52)
    z = to_np(cb.tv_prox(g, z0, H, 600.0, 1e-3, 3))
    want = oracle.tv_prox(g.double().cpu().numpy(), z0.double().cpu().numpy(), H, 600.0, 1e-3, 3)
    assert rel_l2(z, want) <= 20 * 3 * 2.0 ** -24


def test_values_that_are_not_finite_stay_near():
    """NaN and infinities reach one voxel further a step, no more, wherever
    they lie in a box; without clipping a NaN stays one."""
    torch = require_gpu()
    import paper_1002_3675_amd as cb
    shape = (20, 30, 60)
    for at in ((0, 0, 0), (5, 9, 25), (8, 12, 28), (19, 29, 59)):
        for k in (1, 2, 3):
            g, z0 = _case(shape, 53)
            clean = cb.tv_prox(g, z0, H, 600.0, 1e-3, k, nonneg=False)
            bad = z0.clone()
            bad[at] = float("nan")
            got = cb.tv_prox(g, bad, H, 600.0, 1e-3, k, nonneg=False)
            assert torch.isnan(got[at])
            idx = torch.stack(torch.meshgrid(*[torch.arange(n) for n in shape], indexing="ij"))
            far = (idx - torch.tensor(at).view(3, 1, 1, 1)).abs().max(0).values.cuda() > k
            assert torch.equal(got[far], clean[far])

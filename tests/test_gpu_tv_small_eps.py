"""TV steps whose eps^2 is below the smallest float: p = Dz / |Dz| where the
volume is nowhere flat, at the sides of the grid as inside, and zero where it
is flat.  Against the FP64 oracle; tolerance as for the boxes, 20 k 2^-24."""

import numpy as np
import pytest

import oracle

from gpu_util import require_gpu, rel_l2, to_dev, to_np

pytestmark = pytest.mark.gpu

H = np.array([0.9, 1.1, 2.3])


@pytest.mark.parametrize("shape", [(7, 11, 27), (13, 31, 53), (96, 126, 131)])
@pytest.mark.parametrize("nonneg", [True, False])
def test_eps_whose_square_underflows(shape, nonneg):
    require_gpu()
    import paper_1002_3675_amd as cb
    rng = np.random.default_rng(71)
    g, z0 = (rng.uniform(0.01, 0.02, shape).astype(np.float32) for _ in range(2))
    k, step = 3, 1e-5
    z = to_np(cb.tv_prox(to_dev(g), to_dev(z0), H, 600.0, 1e-25, k, step=step, nonneg=nonneg))
    want = oracle.tv_prox(g.astype(np.float64), z0.astype(np.float64), H, 600.0, 1e-25, k,
                          step=step)
    assert (want > 0).all()
    assert rel_l2(z, want) <= 20 * k * 2.0 ** -24


def test_flat_volume_stays():
    torch = require_gpu()
    import paper_1002_3675_amd as cb
    z = torch.full((13, 31, 53), 0.25, device="cuda")
    assert torch.equal(cb.tv_prox(z, z, H, 600.0, 1e-25, 5, step=1e-5, nonneg=False), z)

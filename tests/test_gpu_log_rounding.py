"""The count logarithm is formed in double and rounded once: against the 80-bit
logarithm rounded to float, all elements agree but for those within the
double's error of the middle between two floats.  An error of 5e-16 makes that
2e-8 of the elements; one of 8e-12, as terms in float leave, 1e-4 of them."""

import numpy as np
import pytest

from gpu_util import require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("spread", [0.01, 0.5, 4.0])
def test_logarithms_are_rounded_once(spread):
    torch = require_gpu()
    import paper_1002_3675_amd as cb
    if np.finfo(np.longdouble).nmant < 63:
        pytest.skip("no 80-bit floats")
    rng = np.random.default_rng(98)
    n = 1 << 21
    flat = rng.uniform(2e4, 6e4, n).astype(np.float32)
    counts = (flat * np.exp(rng.normal(0.0, spread, n))).astype(np.float32)
    print("log rounding %g" % spread, flush=True)
    y = cb.log_counts(torch.from_numpy(counts).cuda(), flat=torch.from_numpy(flat).cuda())
    c = np.maximum(counts, np.float32(1.0)).astype(np.longdouble)
    want = np.log(flat.astype(np.longdouble) / c).astype(np.float32)
    assert np.count_nonzero(y.cpu().numpy() != want) <= 2

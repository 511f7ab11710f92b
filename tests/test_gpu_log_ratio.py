"""The logarithm of the count conversion: counts near, far above and far below
the reference, values that take the general path (zero, negative, not finite,
beyond 10^150), lengths that leave a remainder of the four elements a lane,
and arrays off a 16-byte boundary, against the logarithm in extended
precision (of ratios near 1 the one in double keeps too few digits).

Tolerance: the result is within 2^-35 of the logarithm, relative, before it is
rounded to float: half a unit in the last place and 2^-10 of it."""

import math

import numpy as np
import pytest

from gpu_util import require_gpu, to_dev, to_np

pytestmark = pytest.mark.gpu


def _check(got, ref, c):
    with np.errstate(all="ignore"):
        want = np.log(np.asarray(ref, np.longdouble) / c)
        w32 = want.astype(np.float32)
    special = ~np.isfinite(want)
    assert np.array_equal(got[special], w32[special], equal_nan=True)
    g, w = got[~special], want[~special]
    assert np.all(np.abs(g - w) <= (0.5 + 2.0 ** -10) * np.spacing(np.abs(w32[~special])))


@pytest.mark.parametrize("n,shift", [(1, 0), (3, 0), (1023, 0), (4096, 0), (4099, 0), (4099, 1),
                                     (70001, 0)])
def test_log_ratio(n, shift):
    torch = require_gpu()
    import paper_1002_3675_amd as cb
    rng = np.random.default_rng(51)
    print("log of %d ratios" % n, flush=True)
    flat = np.exp(rng.uniform(-30, 60, n)).astype(np.float32)
    c = (flat * np.exp(rng.normal(0, 1, n) * 10.0 ** rng.uniform(-7, 1.3, n))).astype(np.float32)
    sp = np.array([0.0, -1.0, math.inf, -math.inf, math.nan, 1e-40, 1.0], np.float32)
    at = np.arange(0, n, 5)
    flat[at] = sp[at % 7]
    c[at[::3]] = sp[(at[::3] // 5) % 7]
    buf = [torch.empty(n + shift, device="cuda") for _ in range(3)]
    cd, fd, out = (b[shift:] for b in buf)
    cd.copy_(to_dev(c))
    fd.copy_(to_dev(flat))
    for low in (1.0, 1e-20):
        lim = np.where(np.isnan(c), low, np.maximum(c.astype(np.float64), low))
        _check(to_np(cb.log_counts(cd, flat=fd, min_count=low, out=out)).astype(np.float32), flat, lim)
        for i0 in (5e4, 3e-40, 1e200):
            _check(to_np(cb.log_counts(cd, i0=i0, min_count=low, out=out)).astype(np.float32), i0, lim)

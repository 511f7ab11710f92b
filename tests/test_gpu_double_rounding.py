"""The double transpose against sums over 80-bit sample positions.  What it errs
by is the rounding of the rays' increments, 2^-54 of some 300 cells to the
source and a few operations: 1e-14 to 1e-13 of a cell, and of the weights.  A
voxel's samples come from many rays, each with roundings of its own, which
average out; one ray's line used for all of a column's would not.  The bounds
are 2.5% above what the kernel errs by that takes every sample by itself,
3.859e-14 and 3.462e-14 (a column's line: 4.138e-14 in the first case)."""

import math

import numpy as np
import pytest

from workloads import Geometry

from gpu_util import require_gpu

pytestmark = pytest.mark.gpu

L = np.longdouble


def _transpose80(g, r):
    n, h = (g.nx, g.ny, g.nz), [L(x) for x in (g.hx, g.hy, g.hz)]
    step = L(0.5) * min(h)
    x0 = [-L(0.5) * (n[a] - 1) * h[a] for a in range(3)]
    u = (np.arange(g.nu) - L(0.5) * (g.nu - 1)) * L(g.au)
    v = (np.arange(g.nv) - L(0.5) * (g.nv - 1)) * L(g.av)
    U, V = np.meshgrid(u, v)
    inv = 1 / np.sqrt(U * U + V * V + L(g.sdd) ** 2)
    out = np.zeros((g.nz + 2, g.ny + 2, g.nx + 2), L)
    half = 0.5 * math.sqrt(sum(((n[a] + 2) * float(h[a])) ** 2 for a in range(3)))
    for k in range(g.n_views):
        th = L(2.0 * math.pi * k / g.n_views)
        cs, sn = np.cos(th), np.sin(th)
        s = (L(g.sad) * sn, -L(g.sad) * cs, L(0))
        d = ((U * cs - L(g.sdd) * sn) * inv, (U * sn + L(g.sdd) * cs) * inv, V * inv)
        for m in range(int((g.sad - half) / step), int((g.sad + half) / step) + 2):
            q = [(s[a] - x0[a] + L(m) * step * d[a]) / h[a] for a in range(3)]
            f = [np.floor(x) for x in q]
            ok = np.logical_and.reduce([(f[a] >= -1) & (f[a] < n[a]) for a in range(3)])
            if not ok.any():
                continue
            i = [x[ok].astype(int) + 1 for x in f]
            w = [(q[a] - f[a])[ok] for a in range(3)]
            rv = r[k][ok] * step
            for o in range(8):
                p = [w[a] if o >> a & 1 else 1 - w[a] for a in range(3)]
                np.add.at(out, (i[2] + (o >> 2), i[1] + (o >> 1 & 1), i[0] + (o & 1)),
                          p[0] * p[1] * p[2] * rv)
    return out[1:-1, 1:-1, 1:-1]


# three detector rows a cell and more, and fewer
CASES = {"rows": (Geometry(60, 52, 20, 2.0, 2.0, 4.0, 90, 70, 1.8, 1.2, 1000.0, 1500.0, 11), 3.95e-14),
         "rays": (Geometry(40, 44, 30, 2.0, 2.0, 2.0, 80, 60, 1.5, 1.5, 1000.0, 1500.0, 9), 3.55e-14)}


@pytest.mark.parametrize("name", sorted(CASES))
def test_double_transpose_errs_as_its_rays(name):
    torch = require_gpu()
    import paper_1002_3675_amd as cb
    if np.finfo(L).nmant < 63:
        pytest.skip("no 80-bit floats")
    g, bound = CASES[name]
    r = np.random.default_rng(105).standard_normal(g.proj_shape)
    want = _transpose80(g, r.astype(L))
    print("80-bit transpose %s" % name, flush=True)
    f = cb.Plan(g).backproject(torch.from_numpy(r).cuda()).cpu().numpy()
    err = float(np.linalg.norm((f - want).astype(float)) / np.linalg.norm(want.astype(float)))
    print("error %.3e" % err, flush=True)
    assert err <= bound

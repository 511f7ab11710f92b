"""TV steps of grids that are swept, one step a launch: few planes or rows, which
fill little of the boxes that make several steps a launch.  Rows of four and of
other numbers of voxels, arrays that are not 16-byte aligned, planes in several
chunks, against the FP64 oracle, and the time of a single plane.

Tolerance: as for the boxes, 20 k 2^-24 for k steps."""

import numpy as np
import pytest

import oracle

from gpu_util import require_gpu, rel_l2, to_np

pytestmark = pytest.mark.gpu

H = np.array([0.9, 1.1, 2.3])
SHAPES = [(1, 600, 512), (1, 601, 513), (1, 8, 30001), (1, 1, 100000), (2, 512, 512),
          (4, 1024, 1024), (6905, 1, 32), (8999, 2, 28)]


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("aligned", [True, False])
def test_swept_grids_match_oracle(shape, aligned):
    torch = require_gpu()
    import paper_1002_3675_amd as cb
    rng = np.random.default_rng(61)
    g, z0 = (rng.uniform(lo, 0.02, shape).astype(np.float32) for lo in (-0.002, 0.0))

    def dev(x):
        flat = torch.empty(x.size + 1, dtype=torch.float32, device="cuda")
        t = flat[0 if aligned else 1:][:x.size].view(shape)
        t.copy_(torch.from_numpy(x))
        assert (t.data_ptr() % 16 == 0) == aligned
        return t

    print("tv sweeps %s %s" % (shape, aligned), flush=True)
    k = 5
    z = to_np(cb.tv_prox(dev(g), dev(z0), H, 600.0, 1e-3, k, out=dev(z0)))
    want = oracle.tv_prox(g.astype(np.float64), z0.astype(np.float64), H, 600.0, 1e-3, k)
    assert rel_l2(z, want) <= 20 * k * 2.0 ** -24


def test_a_single_plane_takes_a_few_copies_time():
    """A step reads two arrays and writes one: about twice a copy's time.  In
    boxes of twelve planes it took nine times as long."""
    torch = require_gpu()
    import paper_1002_3675_amd as cb
    z = torch.rand((1, 4096, 4096), device="cuda")
    out, n = z.clone(), 24

    def ms(call):
        call()
        a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        a.record()
        call()
        b.record()
        torch.cuda.synchronize()
        return a.elapsed_time(b)

    def copies():
        for _ in range(n):
            out.copy_(z)

    t = ms(copies)
    assert ms(lambda: cb.tv_prox(z, out, H, 600.0, 1e-3, n, out=out)) <= 5 * t


def _steps64(g, z, k, cut):
    """k steps in float64 of a box cut out of a grid; cut[a] = (low, high): whether
    that side of axis a is a cut, k voxels from which the values are not the
    grid's own."""
    import torch
    eps, beta = 1e-3, 600.0
    step = 1.0 / (beta + 4.0 * float(np.sum(H ** -2)) / eps)
    g, z = g.double(), z.double()
    for _ in range(k):
        p = []
        for a, h in ((2, H[0]), (1, H[1]), (0, H[2])):
            d = torch.zeros_like(z)
            m = z.shape[a] - 1
            d.narrow(a, 0, m).copy_((z.narrow(a, 1, m) - z.narrow(a, 0, m)) / h)
            p.append(d)
        norm = torch.sqrt(p[0] ** 2 + p[1] ** 2 + p[2] ** 2 + eps * eps)
        grad = beta * (z - g)
        for (a, h), d in zip(((2, H[0]), (1, H[1]), (0, H[2])), p):
            d = d / norm / h
            m = z.shape[a] - 1
            grad = grad - d
            grad.narrow(a, 1, m).add_(d.narrow(a, 0, m))
        z = (z - step * grad).clamp(min=0.0)
    for a, (low, high) in enumerate(cut):
        z = z.narrow(a, k * low, z.shape[a] - k * (low + high))
    return z


@pytest.mark.parametrize("shape,boxes", [
    # rows beyond the boxes' offsets, planes in two chunks
    ((17, 2, 2 ** 24 + 5), [((12, 17), (0, 2), (0, 300)), ((0, 17), (0, 2), (2 ** 24 - 200, 2 ** 24 + 5))]),
    # and rows that begin beyond 2^31 voxels
    ((1, 129, 2 ** 24 + 1), [((0, 1), (118, 129), (0, 300)),
                             ((0, 1), (118, 129), (2 ** 24 - 200, 2 ** 24 + 1))]),
])
def test_long_rows(shape, boxes):
    """Boxes cut out of the volume at its sides, in float64."""
    torch = require_gpu()
    import paper_1002_3675_amd as cb
    torch.manual_seed(62)
    g, z = (torch.rand(shape, device="cuda").mul_(0.02) for _ in range(2))
    k = 3

    def cut(x, box):
        return x[tuple(slice(*s) for s in box)]

    want = [_steps64(cut(g, b), cut(z, b), k,
                     [(s[0] > 0, s[1] < n) for s, n in zip(b, shape)]) for b in boxes]
    print("tv sweep of long rows %s" % (shape,), flush=True)
    cb.tv_prox(g, z, H, 600.0, 1e-3, k, out=z)
    for b, w in zip(boxes, want):
        inner = tuple(slice(s[0] + k * (s[0] > 0), s[1] - k * (s[1] < n)) for s, n in zip(b, shape))
        assert rel_l2(to_np(z[inner]), to_np(w)) <= 20 * k * 2.0 ** -24

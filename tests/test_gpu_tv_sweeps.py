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

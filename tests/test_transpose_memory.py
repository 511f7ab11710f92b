"""Device memory of a solve: the transpose's tables of bricks' views take no more
than a quarter of 64 bytes per brick and view, or 8 GiB where that is more."""

import paper_1002_3675_amd as cb

LEAST = 8 << 30


def _rest(g):
    """Bytes of a one-level matched solve without the table, as the steps need
    them: data and residual, f, g, z, padded volume, eight cell sums, ray table."""
    meas, vox = g.nu * g.nv * g.n_views, g.nx * g.ny * g.nz
    cells = 8 * (-(-(g.nx + 1) // 32) * 32) * (g.ny + 1) * (g.nz + 1)
    pad = (g.nx + 2) * (g.ny + 2) * (g.nz + 2)
    return 4 * (2 * meas + 3 * vox + pad + cells) + 24 * meas


def _bricks(g):
    return -(-(g.nx + 1) // 16) * -(-(g.ny + 1) // 16) * (g.nz + 1)


def test_large_scans_keep_a_quarter():
    for g in (cb.Geometry(512, 512, 512, 0.5, 0.5, 0.5, 1024, 1024, 0.5, 0.5, 1000.0, 1500.0, 720),
              cb.Geometry(760, 760, 760, 0.3, 0.3, 0.3, 1000, 1000, 0.5, 0.5, 1000.0, 1500.0, 2000)):
        got = cb.footprint(g, cb.FbsParams(iters=(10,), beta=(500.0,)))
        table = 16 * _bricks(g) * g.n_views
        assert 4 * table > LEAST
        # partial sums and alignment are far below a hundredth of the table
        assert _rest(g) + 0.99 * table <= got <= _rest(g) + 1.01 * max(table, LEAST)


def test_other_scans_keep_all():
    g = cb.Geometry(512, 512, 70, 0.88, 0.88, 2.5, 512, 384, 0.776, 0.776, 1000.0, 1500.0, 40)
    table = 64 * _bricks(g) * g.n_views
    assert table < LEAST
    assert cb.footprint(g, cb.FbsParams(iters=(10,), beta=(500.0,))) >= _rest(g) + table

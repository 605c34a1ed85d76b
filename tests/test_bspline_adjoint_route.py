"""The rule that sends the control-grid adjoint's z and y sums plane by plane or through
a pass each (ctaug::bspline_adj_by_planes, host code): fields and grids at which one of
the two was measured to be at least 1.3 times faster.  On the GPU, fields that go plane
by plane with every grid class against the oracle's FP64 sums, in one to three chunks of
rows and up to three segments of z, and the same bits twice."""
import ctypes

import numpy as np
import pytest

from paper_1811_11226_amd import _lib


class Geom(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int32) for n in ("ox", "oy", "oz", "gx", "gy", "gz")] + \
               [(n, ctypes.c_float) for n in ("inv_hx", "inv_hy", "inv_hz")]


def _by_planes(dims, grid):
    rule = _lib.load()._ZN5ctaug21bspline_adj_by_planesERKNS_11BsplineGeomEb
    rule.restype = ctypes.c_bool
    return rule(ctypes.byref(Geom(*dims, *grid)), ctypes.c_bool(dims[2] % 4 == 0))


PASSES = [((1, 2000, 2000), (8, 8, 8)), ((4, 512, 512), (16, 16, 16)), ((16, 512, 512), (32, 32, 32)),
          ((40, 300, 300), (32, 32, 32)), ((40, 300, 300), (64, 64, 64)), ((30, 33, 35), (64, 64, 64)),
          ((8, 4000, 8), (64, 64, 64)), ((96, 96, 96), (24, 24, 24)), ((2000, 8, 8), (64, 64, 64)),
          ((20000, 1, 4), (24, 24, 24)), ((24, 256, 256), (8, 64, 4))]
PLANES = [((128, 128, 128), (8, 8, 8)), ((117, 130, 151), (12, 12, 12)), ((256, 256, 256), (9, 9, 9)),
          ((48, 48, 48), (5, 5, 5)), ((8, 8, 4000), (8, 8, 8)), ((8, 4000, 8), (8, 8, 8)),
          ((200, 190, 210), (16, 16, 16)), ((512, 512, 64), (32, 32, 32)), ((40, 300, 300), (8, 8, 8)),
          ((64, 64, 301), (64, 64, 64)), ((30, 33, 35), (16, 16, 16))]


@pytest.mark.parametrize("dims,grid", PASSES)
def test_passes(dims, grid):
    assert not _by_planes(dims, grid)


@pytest.mark.parametrize("dims,grid", PLANES)
def test_planes(dims, grid):
    assert _by_planes(dims, grid)


@pytest.mark.gpu
@pytest.mark.parametrize("grid", [(4, 4, 4), (8, 8, 8), (5, 9, 8), (6, 16, 16), (4, 17, 16),
                                  (7, 64, 16), (5, 6, 17), (4, 16, 64), (64, 64, 64)])
@pytest.mark.parametrize("dims", [(6, 130, 1001), (8, 70, 1401), (16, 64, 401), (5, 1, 1030)])
def test_adjoint_by_planes(dims, grid):
    import torch

    import oracle
    import paper_1811_11226_amd as ctaug
    if not _by_planes(dims, grid):
        assert dims[1] == 130 and grid[2] == 64        # the only ones left to the passes
    rng = np.random.default_rng(sum(grid) + sum(dims))
    g = rng.normal(0, 1, (3,) + dims).astype(np.float32)
    out = ctaug.bspline_upsample_adjoint(torch.from_numpy(g).cuda(), grid)
    again = ctaug.bspline_upsample_adjoint(torch.from_numpy(g).cuda(), grid)
    assert torch.equal(out, again)
    ref = oracle.bspline_adjoint(g.astype(np.float64), grid)
    # FP32: each term's weights carry about 20 roundings and the cell coordinate two
    # of p / h; a z sum of m terms at most m more; bounded by the sum of |terms|
    mag = oracle.bspline_adjoint(np.abs(g).astype(np.float64), grid)
    tol = (60 + 2 * dims[2] + 12 * max(grid) + max(dims)) * 2.0 ** -24
    assert np.all(np.abs(out.cpu().numpy() - ref) <= tol * mag + 64 * 2.0 ** -24 * mag.max())


# More planes than the first dimension of the grid holds, plane by plane.
@pytest.mark.gpu
def test_many_planes():
    import torch

    import oracle
    import paper_1811_11226_amd as ctaug
    dims, grid = (21846, 24, 28), (4, 4, 4)
    assert _by_planes(dims, grid)
    g = np.random.default_rng(2).normal(0, 1, (3,) + dims).astype(np.float32)
    out = ctaug.bspline_upsample_adjoint(torch.from_numpy(g).cuda(), grid).cpu().numpy()
    ref = oracle.bspline_adjoint(g, grid)
    assert np.linalg.norm(out - ref) <= 1e-4 * np.linalg.norm(ref)

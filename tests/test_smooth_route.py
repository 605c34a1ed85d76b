"""The rule that sends a smoothing to the one fused pass or to a pass per axis
(ctaug::smooth_fused_ok, host code): sizes at which one of the two was measured to be
at least 1.2 times faster, each radius, single axes, and radii and planes that only
the passes take.  On the GPU, volumes that take the fused pass at the edges of its
tiles and x chunks give the bits of the axes smoothed one call at a time."""
import ctypes

import numpy as np
import pytest

from paper_1811_11226_amd import _lib

# sigma of a radius R: 3 sigma / sqrt(2) + 0.5 in [R, R + 1)
SIGMA = {0: 0.0, 1: 0.5, 2: 1.0, 3: 1.4, 4: 1.9}

PASSES = [((32, 32, 32), (2, 2, 2)), ((32, 32, 32), (4, 4, 4)), ((64, 64, 64), (3, 3, 3)),
          ((64, 64, 64), (4, 4, 4)), ((96, 96, 96), (3, 3, 3)), ((128, 128, 60), (3, 3, 3)),
          ((128, 128, 60), (4, 4, 4)), ((128, 128, 128), (3, 3, 3)), ((160, 160, 100), (4, 4, 4)),
          ((128, 128, 128), (0, 0, 2)), ((192, 192, 96), (2, 0, 0)), ((40, 48, 36), (3, 3, 3)),
          ((1000, 8, 8), (4, 4, 4)), ((512, 512, 320), (2, 5, 1)), ((1, 32768, 16384), (1, 1, 1))]
FUSED = [((64, 64, 64), (1, 1, 1)), ((32, 32, 32), (1, 1, 1)), ((128, 128, 60), (2, 2, 2)),
         ((192, 192, 96), (3, 3, 3)), ((160, 160, 100), (2, 2, 2)), ((256, 256, 120), (4, 4, 4)),
         ((512, 512, 320), (2, 2, 2)), ((512, 512, 320), (4, 4, 4)), ((512, 512, 1), (4, 4, 4)),
         ((16, 512, 512), (4, 4, 4)), ((512, 16, 512), (3, 3, 3)), ((300, 300, 60), (0, 0, 2)),
         ((384, 384, 200), (1, 0, 0)), ((8, 1000, 8), (3, 3, 3))]


def _fused(dims, radii):
    rule = _lib.load()._ZN5ctaug15smooth_fused_okEPKiS1_
    rule.restype = ctypes.c_bool
    return rule((ctypes.c_int32 * 3)(*radii), (ctypes.c_int32 * 3)(*dims))


@pytest.mark.parametrize("dims,radii", PASSES)
def test_passes(dims, radii):
    assert not _fused(dims, radii)


@pytest.mark.parametrize("dims,radii", FUSED)
def test_fused(dims, radii):
    assert _fused(dims, radii)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [np.float32, np.int16])
@pytest.mark.parametrize("dims,radii", [((50, 65, 121), (1, 1, 1)), ((6, 65, 121), (3, 3, 3)),
                                        ((41, 250, 130), (2, 2, 2)), ((57, 400, 121), (3, 2, 3)),
                                        ((72, 500, 130), (4, 4, 4)), ((7, 33, 249), (4, 1, 4)),
                                        ((4, 31, 124), (0, 3, 2)), ((3, 2, 2), (4, 4, 4)),
                                        ((300, 201, 60), (0, 0, 2)), ((50, 400, 241), (2, 0, 1))])
def test_fused_edges(dims, radii, dtype):
    import torch

    import paper_1811_11226_amd as ctaug
    assert _fused(dims, radii)
    rng = np.random.default_rng(sum(dims) + sum(radii))
    v = torch.from_numpy(np.round(rng.uniform(-1000, 2000, dims)).astype(dtype)).cuda()
    out = ctaug.gaussian_smooth(v, [SIGMA[r] for r in radii])
    step = v.float()
    for axis in range(3):
        step = ctaug.gaussian_smooth(step, [SIGMA[radii[a]] if a == axis else 0.0 for a in range(3)])
    assert torch.equal(out, step)


# Even z extents from addresses that do not allow a lane's two voxels at once.
@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["float32", "int16"])
@pytest.mark.parametrize("off_in,off_out", [(1, 0), (0, 1), (1, 1), (2, 2)])
def test_fused_misaligned_pairs(dtype, off_in, off_out):
    import torch

    import paper_1811_11226_amd as ctaug
    dims, radii = (6, 34, 126), (2, 1, 3)
    assert _fused(dims, radii)
    sigma = [SIGMA[r] for r in radii]
    n = dims[0] * dims[1] * dims[2]
    flat = torch.randint(-1000, 2000, (n + 2,), device="cuda").to(getattr(torch, dtype))
    v = flat[off_in:off_in + n].view(dims)
    out = torch.full((n + 4,), 7.0, device="cuda")
    ctaug.gaussian_smooth(v, sigma, out=out[off_out:off_out + n].view(dims))
    ref = ctaug.gaussian_smooth(v.clone(), sigma)
    assert torch.equal(out[off_out:off_out + n].view(dims), ref)
    assert (out[:off_out] == 7.0).all() and (out[off_out + n:] == 7.0).all()

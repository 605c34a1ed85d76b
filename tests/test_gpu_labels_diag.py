"""Labels under diagonal maps (a plane's, a row's and a column's cells apart) against
the oracle: extents around the 4, 8 and 16 voxels a lane takes, rows past one
pass, odd (unaligned) rows, reflections, shifts past both faces, ties, strided
inputs, one-voxel axes, and maps a hair off the diagonal (the general kernel)."""
import numpy as np
import pytest
import torch

import oracle
import paper_1811_11226_amd as ctaug

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nout", [(5, 33, 4), (6, 17, 255), (3, 21, 256), (4, 5, 257), (7, 3, 511),
                                  (2, 9, 512), (3, 4, 513), (2, 3, 1025), (1, 1, 1), (40, 130, 31)])
@pytest.mark.parametrize("scale,shift", [((0.31, 0.44, 0.2), (0.0, 0.0, 0.0)),
                                         ((1.0, 1.0, 1.0), (0.5, -0.5, 1.5)),
                                         ((-0.5, 0.7, -0.25), (9.0, -3.0, 30.0)),
                                         ((2.0, 0.0, 3.0), (-4.0, 2.49, -7.0)),
                                         ((1e9, 1.0, 1.0), (0.0, 0.0, 0.0))])
def test_diagonal_labels(nout, scale, shift):
    rng = np.random.default_rng(sum(nout))
    whole = rng.integers(-5, 6, (21, 26, 47)).astype(np.int8)
    lbl = whole[2:18, 3:23, 4:44]
    M = np.concatenate([np.diag(scale), np.array(shift)[:, None]], axis=1).astype(np.float32)
    img = np.zeros(lbl.shape, dtype=np.float32)
    t = torch.from_numpy(whole).cuda()[2:18, 3:23, 4:44]
    for off in (0.0, 1e-30):
        M[0, 1] = off
        _, ref = oracle.warp(img, M, nout, lbl=np.ascontiguousarray(lbl), label_fill=-9)
        out = torch.full((int(np.prod(nout)) + 3,), 77, dtype=torch.int8, device="cuda")
        view = out[1:1 + int(np.prod(nout))].view(nout)       # rows at any alignment
        ctaug.warp_labels(t, M, label_fill=-9, lbl_out=view)
        got = out.cpu().numpy()
        assert np.array_equal(got[1:-2].reshape(nout), ref)
        assert got[0] == 77 and got[-1] == 77 and got[-2] == 77

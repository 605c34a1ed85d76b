"""Labels under diagonal maps whose rows are walked in segments (rows past 512 voxels,
rows enough), and such rows in volumes too thin for it, against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_1811_11226_amd as ctaug

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nout", [(64, 64, 513), (33, 125, 767), (32, 128, 1030), (257, 13, 769),
                                  (64, 60, 515), (2, 9, 1500)])
@pytest.mark.parametrize("scale,shift", [((0.31, 0.44, 0.06), (0.0, 0.0, 0.0)),
                                         ((-0.25, 0.16, -0.04), (9.0, -3.0, 39.0)),
                                         ((1.0, 1.0, 1.0), (-7.0, 0.5, -480.5))])
def test_segments(nout, scale, shift):
    rng = np.random.default_rng(sum(nout))
    lbl = rng.integers(-5, 6, (16, 20, 40)).astype(np.int8)
    M = np.concatenate([np.diag(scale), np.array(shift)[:, None]], axis=1).astype(np.float32)
    _, ref = oracle.warp(np.zeros(lbl.shape, np.float32), M, nout, lbl=lbl, label_fill=-9,
                         want_img=False)
    n = int(np.prod(nout))
    out = torch.full((n + 3,), 77, dtype=torch.int8, device="cuda")
    ctaug.warp_labels(torch.from_numpy(lbl).cuda(), M, label_fill=-9,
                      lbl_out=out[1:1 + n].view(nout))            # rows at any alignment
    got = out.cpu().numpy()
    assert np.array_equal(got[1:-2].reshape(nout), ref)
    assert got[0] == 77 and got[-1] == 77 and got[-2] == 77

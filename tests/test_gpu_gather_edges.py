"""Tiles that are gathered from memory and reach past the output's end, whose class is that
of voxels inside it: thin outputs, remainders of 1 to 3 voxels of a run and of 1 of a tile,
with the samples just inside, on and past the volume's faces; single calls and plans."""
import numpy as np
import pytest
import torch

import oracle
import paper_1811_11226_amd as ctaug

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nout", [(9, 17, 12), (5, 9, 1), (8, 8, 13), (4, 3, 18), (33, 9, 33),
                                  (6, 40, 35), (1, 1, 50)])
@pytest.mark.parametrize("scale", [(2.6, 2.6, 13.0), (-6.0, 5.0, 7.0)])
@pytest.mark.parametrize("rim", [0, 1])
@pytest.mark.parametrize("shift", [0.0, -0.75, 0.75])
@pytest.mark.parametrize("dtype", [np.float32, np.int16])
def test_gather_edges(nout, scale, rim, shift, dtype):
    # samples from the first cell's centre to the last one's where rim = 0
    nin = tuple(int(np.ceil(abs(s) * (o - 1))) + 1 + 2 * rim for s, o in zip(scale, nout))
    rng = np.random.default_rng(sum(nin))
    img = rng.integers(-1000, 2000, nin).astype(dtype)
    lbl = rng.integers(1, 6, nin).astype(np.int8)
    M = np.zeros((3, 4), np.float32)
    for i in range(3):
        M[i, i] = scale[i]
        M[i, 3] = (rim if scale[i] > 0 else nin[i] - 1 - rim) + shift
    ref, lref = oracle.warp(img, M, nout, lbl=lbl, fill=-1000.0, label_fill=-3)
    ti, tl = torch.from_numpy(img).cuda(), torch.from_numpy(lbl).cuda()
    out, lout = ctaug.warp_affine(ti, M, lbl=tl, fill=-1000.0, label_fill=-3, out_dim=nout)
    assert np.array_equal(lout.cpu().numpy(), lref)
    assert np.all(np.abs(out.cpu().numpy() - ref) <= 1e-5 * np.maximum(np.abs(ref), 1000.0))
    for tile in ((16, 16, 16), (4, 8, 4), (2, 8, 128)):
        o2, l2 = torch.full_like(out, 7.0), torch.full_like(lout, 7)
        job = ctaug.make_job(ti, M, o2, lbl=tl, lbl_out=l2, fill=-1000.0, label_fill=-3)
        plan = ctaug.BatchPlan([job], tile=tile, lds_cells=-1)
        plan.launch()
        torch.cuda.synchronize()
        assert torch.equal(o2, out) and torch.equal(l2, lout), tile
        plan.close()

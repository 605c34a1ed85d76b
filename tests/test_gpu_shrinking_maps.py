"""Shrinking maps at and around the lines where windows are no longer staged (z runs that
keep to their rows, small turns, sub-tiles of 4 voxels along z), against the oracle, and
plans against single calls bit for bit."""
import numpy as np
import pytest
import torch

import oracle
import paper_1811_11226_amd as ctaug
from test_gpu_fwd_windows import _map, _rot

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nout", [(33, 31, 40), (17, 20, 16), (20, 18, 5), (24, 30, 4), (9, 40, 33)])
@pytest.mark.parametrize("scale", [1.8, 2.1, 2.5, 3.2])
@pytest.mark.parametrize("turn", [0.0, 0.002, 0.02, 0.3])
@pytest.mark.parametrize("dtype", [np.float32, np.int16])
def test_shrinking(nout, scale, turn, dtype):
    nin = tuple(int(v * scale) + 1 for v in nout)
    rng = np.random.default_rng(sum(nin))
    img = rng.integers(-1000, 2000, nin).astype(dtype)
    lbl = rng.integers(1, 6, nin).astype(np.int8)
    M = _map(scale * _rot(turn, -turn, 0.7 * turn), nin, nout)
    ref, lref = oracle.warp(img, M, nout, lbl=lbl, fill=-1000.0, label_fill=-3)
    ti, tl = torch.from_numpy(img).cuda(), torch.from_numpy(lbl).cuda()
    out, lout = ctaug.warp_affine(ti, M, lbl=tl, fill=-1000.0, label_fill=-3, out_dim=nout)
    assert np.array_equal(lout.cpu().numpy(), lref)
    assert np.all(np.abs(out.cpu().numpy() - ref) <= 1e-5 * np.maximum(np.abs(ref), 1000.0))
    for tile, cells in [(None, 0), ((16, 16, 16), 0), ((4, 8, 4), 3000), ((8, 16, 16), 15000)]:
        o2, l2 = torch.full_like(out, 7.0), torch.full_like(lout, 7)
        job = ctaug.make_job(ti, M, o2, lbl=tl, lbl_out=l2, fill=-1000.0, label_fill=-3)
        plan = ctaug.BatchPlan([job], tile=tile, lds_cells=cells)
        plan.launch()
        torch.cuda.synchronize()
        assert torch.equal(o2, out) and torch.equal(l2, lout), (tile, cells)
        plan.close()


# Tiles past the reservation inside the volume (their cells gathered without tests), over
# its faces, and outside it.
@pytest.mark.parametrize("nout", [(33, 31, 40), (16, 17, 19)])
@pytest.mark.parametrize("scale,std", [(3.0, 1.0), (4.5, 6.0), (0.9, 25.0)])
@pytest.mark.parametrize("dtype", [np.float32, np.int16])
def test_displaced(nout, scale, std, dtype):
    nin = tuple(int(v * max(scale, 2.0)) + 1 for v in nout)
    rng = np.random.default_rng(sum(nin))
    img = rng.integers(-1000, 2000, nin).astype(dtype)
    lbl = rng.integers(1, 6, nin).astype(np.int8)
    M = _map(scale * _rot(0.1, -0.2, 0.15), nin, nout)
    ctrl = rng.normal(0, std, (3, 6, 5, 7)).astype(np.float32)
    u = oracle.bspline_upsample_f32(ctrl, nout)
    ref, lref = oracle.warp(img, M, nout, lbl=lbl, disp=u, fill=-1000.0, label_fill=-3)
    t = lambda a: torch.from_numpy(a).cuda()  # noqa: E731
    for out, lout in (ctaug.warp_displacement(t(img), M, t(u), lbl=t(lbl), fill=-1000.0,
                                              label_fill=-3),
                      ctaug.warp_bspline(t(img), M, t(ctrl), lbl=t(lbl), fill=-1000.0,
                                         label_fill=-3, out_dim=nout)):
        assert np.array_equal(lout.cpu().numpy(), lref)
        assert np.all(np.abs(out.cpu().numpy() - ref) <= 1e-5 * np.maximum(np.abs(ref), 1000.0))

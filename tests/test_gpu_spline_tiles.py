"""The displacement of a tile evaluated in the warp: windows of 4 to 8 controls per
axis, wider ones along each axis (profiles one by one, or every voxel its own), and
cells that change inside a thread's run, bit for bit against the upsampled field;
footprints past the reservation; one- and two-voxel axes."""
import numpy as np
import pytest
import torch

import oracle
import paper_1811_11226_amd as ctaug

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("grid", [(4, 4, 4), (5, 7, 6), (8, 8, 8), (12, 9, 21), (30, 6, 5),
                                  (5, 33, 9), (6, 5, 40), (25, 28, 31)])
@pytest.mark.parametrize("dims", [(17, 9, 33), (8, 8, 16), (40, 23, 35), (1, 5, 2), (2, 1, 19)])
def test_tile_field_equals_upsampled(grid, dims):
    rng = np.random.default_rng(sum(grid) + sum(dims))
    img = torch.from_numpy(rng.normal(0, 300, (30, 28, 34)).astype(np.float32)).cuda()
    lbl = torch.from_numpy(rng.integers(0, 6, img.shape).astype(np.int8)).cuda()
    ctrl = torch.from_numpy(rng.normal(0, 2, (3,) + grid).astype(np.float32)).cuda()
    M = np.eye(3, 4, dtype=np.float32)
    M[:, 3] = (3.3, -1.2, 4.6)
    out, lout = ctaug.warp_bspline(img, M, ctrl, lbl=lbl, out_dim=dims, fill=-7.0, label_fill=-1)
    u = ctaug.bspline_upsample(ctrl, dims)
    ref, lref = ctaug.warp_displacement(img, M, u, lbl=lbl, fill=-7.0, label_fill=-1)
    assert torch.equal(out, ref) and torch.equal(lout, lref)
    o2, l2 = torch.empty_like(out), torch.empty_like(lout)
    plan = ctaug.BatchPlan([ctaug.make_job(img, M, o2, lbl=lbl, lbl_out=l2, fill=-7.0,
                                           label_fill=-1, ctrl=ctrl)])
    plan.launch()
    torch.cuda.synchronize()
    assert torch.equal(o2, out) and torch.equal(l2, lout)
    plan.close()


@pytest.mark.parametrize("std", [1.0, 8.0, 60.0])
def test_tiles_past_the_reservation_gather_the_same(std):
    """Fields from gentle to wild: staged and gathered tiles meet in one volume; the
    identity map with an integer field is an exact shift."""
    rng = np.random.default_rng(int(std))
    n = (40, 33, 50)
    img_np = rng.integers(-1000, 2000, n).astype(np.int16)
    d = np.rint(rng.normal(0, std, (3,) + n)).astype(np.float32)
    out, _ = ctaug.warp_displacement(torch.from_numpy(img_np).cuda(), np.eye(3, 4), torch.from_numpy(
        d).cuda(), fill=9.0)
    at = [g + d[i].astype(np.int64) for i, g in enumerate(np.meshgrid(
        *[np.arange(v) for v in n], indexing="ij"))]
    ok = np.all([(a >= 0) & (a < v) for a, v in zip(at, n)], axis=0)
    ref = np.where(ok, img_np[tuple(np.clip(a, 0, v - 1) for a, v in zip(at, n))], 9.0)
    assert np.array_equal(out.cpu().numpy(), ref.astype(np.float32))


# Upsampled fields at the edges of rows of 8 and of z runs of 256, as the parity-mode
# field.
@pytest.mark.parametrize("dims,grid", [((1, 1, 1), (4, 4, 4)), ((3, 7, 63), (5, 4, 9)),
                                       ((2, 8, 64), (4, 6, 64)), ((5, 9, 257), (6, 5, 12)),
                                       ((2, 17, 255), (4, 64, 5)), ((4, 16, 512), (64, 7, 30))])
def test_upsampling_rows(dims, grid):
    rng = np.random.default_rng(sum(dims))
    c = rng.normal(0, 4, (3,) + grid).astype(np.float32)
    u = ctaug.bspline_upsample(torch.from_numpy(c).cuda(), dims).cpu().numpy()
    assert np.array_equal(u, oracle.bspline_upsample_f32(c, dims))

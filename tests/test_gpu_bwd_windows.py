"""The adjoints where their windows, flush and groups can go wrong, against the
oracle: thin volumes, footprints past every face, maps past the 32-bit bound,
past the windows' reservation and singular ones, groups of one tile up to more
than the partial rows hold, strided inputs, and batches of uneven jobs."""
import numpy as np
import pytest
import torch

import oracle
import paper_1811_11226_amd as ctaug
from paper_1811_11226_amd import ops
from test_gpu_fwd_windows import MAPS, _map

pytestmark = pytest.mark.gpu


def _close(got, ref, what):
    n = np.linalg.norm(ref)
    assert np.linalg.norm(got.astype(np.float64) - ref) <= 1e-4 * max(n, 1e-30), what


@pytest.mark.parametrize("name", sorted(MAPS))
@pytest.mark.parametrize("nin,nout", [((37, 41, 39), (33, 35, 36)), ((20, 3, 40), (18, 17, 21)),
                                      ((33, 30, 3), (20, 18, 40)), ((1, 34, 5), (16, 16, 16)),
                                      ((9, 8, 7), (40, 33, 37)), ((60, 50, 70), (8, 8, 16))])
@pytest.mark.parametrize("dtype", [np.float32, np.int16])
def test_affine_adjoint(name, nin, nout, dtype):
    rng = np.random.default_rng(9)
    whole = rng.integers(-1000, 2000, tuple(v + 3 for v in nin)).astype(dtype)
    box = tuple(slice(1, 1 + v) for v in nin)
    g = rng.normal(0, 1, nout).astype(np.float32)
    M = _map(MAPS[name], nin, nout)
    r_img, r_M, _ = oracle.warp_backward(np.ascontiguousarray(whole[box]), M, g, fill=-1000.0)
    img = torch.from_numpy(whole).cuda()[box]
    g_img, g_M = ctaug.warp_affine_backward(img, M, torch.from_numpy(g).cuda(), fill=-1000.0)
    only, _ = ctaug.warp_affine_backward(img, M, torch.from_numpy(g).cuda(), fill=-1000.0,
                                         want_M=False)
    _close(g_img.cpu().numpy(), r_img, "g_img")
    _close(only.cpu().numpy(), r_img, "g_img alone")
    _close(g_M.cpu().numpy(), r_M, "g_M")


def test_more_tiles_than_rows():
    """A long output: 2500 tiles, two per group past the 2048 rows of partials; grad_M
    twice with the same bits."""
    rng = np.random.default_rng(10)
    img = rng.normal(0, 100, (300, 9, 40)).astype(np.float32)
    nout = (8 * 2500, 3, 10)
    g = rng.normal(0, 1, nout).astype(np.float32)
    M = np.array([[0.0149, 0.1, 0, 0.3], [0, 1.2, 0.2, 0.4], [0.0001, 0, 1.1, 2.2]], np.float32)
    r_img, r_M, _ = oracle.warp_backward(img, M, g)
    t, tg = torch.from_numpy(img).cuda(), torch.from_numpy(g).cuda()
    g_img, g_M = ctaug.warp_affine_backward(t, M, tg)
    _close(g_img.cpu().numpy(), r_img, "g_img")
    _close(g_M.cpu().numpy(), r_M, "g_M")
    assert torch.equal(ctaug.warp_affine_backward(t, M, tg)[1], g_M)
    gi, gm = torch.zeros_like(t), torch.zeros(12, dtype=torch.float64, device="cuda")
    ops.warp_affine_backward_noalloc(t, M, tg, grad_img=gi, grad_M=gm)
    assert torch.equal(gm, g_M)


# Windows with rows of more cells than a wave has lanes: along z 9 and 17 input
# voxels per output voxel, in the interior and over the volume's ends.
@pytest.mark.parametrize("nz,scale,shift", [(150, 9.0, 2.0), (150, 9.5, -9.0), (280, 17.0, 3.0),
                                            (262, 17.0, -2.5)])
def test_rows_past_a_wave(nz, scale, shift):
    rng = np.random.default_rng(nz)
    nin, nout = (9, 7, nz), (8, 5, 16)
    img = rng.integers(-1000, 2000, nin).astype(np.float32)
    g = rng.normal(0, 1, nout).astype(np.float32)
    M = np.array([[1, 0, 0, 0.25], [0, 1, 0, 0.5], [0, 0, scale, shift]], np.float32)
    r_img, r_M, _ = oracle.warp_backward(img, M, g, fill=-1000.0)
    g_img, g_M = ctaug.warp_affine_backward(torch.from_numpy(img).cuda(), M,
                                            torch.from_numpy(g).cuda(), fill=-1000.0)
    _close(g_img.cpu().numpy(), r_img, "g_img")
    _close(g_M.cpu().numpy(), r_M, "g_M")


@pytest.mark.parametrize("n", [1, 3, 9])
def test_batches_of_uneven_jobs(n):
    rng = np.random.default_rng(n)
    jobs, refs = [], []
    for i in range(n):
        nin = tuple(int(v) for v in rng.integers(4, 60, 3))
        nout = tuple(int(v) for v in rng.integers(1, 70, 3))
        img = rng.integers(-1000, 2000, nin).astype(np.float32)
        g = rng.normal(0, 1, nout).astype(np.float32)
        M = _map(list(MAPS.values())[i % len(MAPS)], nin, nout)
        refs.append(oracle.warp_backward(img, M, g, fill=-1000.0)[:2])
        gi = torch.zeros(nin, device="cuda")
        gm = torch.full((12,), np.nan, dtype=torch.float64, device="cuda")
        jobs.append((ops.make_bwd_job(torch.from_numpy(img).cuda(), M, torch.from_numpy(g).cuda(),
                                      gi, gm if i % 3 != 1 else None, fill=-1000.0), gi, gm, i))
    ops.warp_affine_backward_batch([j[0] for j in jobs])
    for (_, gi, gm, i), (r_img, r_M) in zip(jobs, refs):
        _close(gi.cpu().numpy(), r_img, f"g_img {i}")
        if i % 3 != 1:
            _close(gm.cpu().numpy(), r_M, f"g_M {i}")

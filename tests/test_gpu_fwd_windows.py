"""The forward warps' footprint windows against the oracle where they can go
wrong: volumes thinner than a quad, windows that reach past every face, maps that
shrink or stretch past what the quad test admits, singular maps, sub-tiles of
every size, coordinates too large for LDS windows, and non-finite voxels and
displacements at the guard."""
import numpy as np
import pytest
import torch

import oracle
import paper_1811_11226_amd as ctaug

pytestmark = pytest.mark.gpu


def _rot(ax, ay, az):
    c, s = np.cos([ax, ay, az]), np.sin([ax, ay, az])
    rx = np.array([[1, 0, 0], [0, c[0], -s[0]], [0, s[0], c[0]]])
    ry = np.array([[c[1], 0, s[1]], [0, 1, 0], [-s[1], 0, c[1]]])
    rz = np.array([[c[2], -s[2], 0], [s[2], c[2], 0], [0, 0, 1]])
    return rz @ ry @ rx


def _map(A, nin, nout, shift=(0.3, -0.7, 0.45)):
    ci, co = (np.array(nin) - 1) / 2, (np.array(nout) - 1) / 2
    return np.concatenate([A, (ci + shift - A @ co)[:, None]], axis=1).astype(np.float32)


R = _rot(0.4, -0.3, 0.5)
MAPS = {"rotation": R, "reflected": R @ np.diag([-1.0, 1.0, -1.0]), "shrink": 0.1 * R,
        "stretch": 2.7 * R, "worst": 1.2 * _rot(0.52, 0.52, 0.52),
        "singular": R @ np.diag([1.0, 0.0, 1.0]), "sheared": R @ np.array(
            [[1, 6.0, 0], [0, 1, 0], [0, 0, 1]]), "zero": np.zeros((3, 3))}


@pytest.mark.parametrize("name", sorted(MAPS))
@pytest.mark.parametrize("nin,nout", [((37, 41, 39), (33, 35, 36)), ((20, 3, 40), (18, 17, 21)),
                                      ((33, 30, 3), (20, 18, 40)), ((1, 34, 5), (16, 16, 16)),
                                      ((26, 24, 4), (31, 9, 44)), ((9, 8, 7), (40, 33, 37))])
@pytest.mark.parametrize("dtype", [np.float32, np.int16])
def test_windows(name, nin, nout, dtype):
    rng = np.random.default_rng(5)
    img = rng.integers(-1000, 2000, nin).astype(dtype)
    lbl = rng.integers(1, 6, nin).astype(np.int8)
    M = _map(MAPS[name], nin, nout)
    ref, lref = oracle.warp(img, M, nout, lbl=lbl, fill=-1000.0, label_fill=-3)
    ti, tl = torch.from_numpy(img).cuda(), torch.from_numpy(lbl).cuda()
    out, lout = ctaug.warp_affine(ti, M, lbl=tl, fill=-1000.0, label_fill=-3, out_dim=nout)
    assert np.array_equal(lout.cpu().numpy(), lref)
    assert np.all(np.abs(out.cpu().numpy() - ref) <= 1e-5 * np.maximum(np.abs(ref), 1000.0))
    # the same bits from every tile, reservation and cell format
    for tile, cells, fmt in [((16, 16, 16), 4096, 0), ((8, 8, 16), 15000, 0), ((16, 16, 64), 9000, 1),
                             ((4, 4, 4), 2000, 0), ((8, 16, 32), -1, 0)]:
        if fmt and dtype != np.int16:
            continue
        o2, l2 = torch.full_like(out, 7.0), torch.full_like(lout, 7)
        job = ctaug.make_job(ti, M, o2, lbl=tl, lbl_out=l2, fill=-1000.0, label_fill=-3)
        plan = ctaug.BatchPlan([job], tile=tile, lds_cells=cells, lds_format=fmt)
        plan.launch()
        torch.cuda.synchronize()
        assert torch.equal(o2, out) and torch.equal(l2, lout), (tile, cells, fmt)
        plan.close()


# Windows past every reservation: cells gathered in pairs along z, in tiles by the
# output's z extent.
@pytest.mark.parametrize("nin,nout", [((90, 80, 150), (9, 7, 17)), ((70, 75, 1), (6, 9, 16)),
                                      ((81, 64, 2), (9, 8, 1)), ((60, 66, 3), (5, 6, 66)),
                                      ((40, 90, 300), (3, 10, 130)), ((64, 50, 140), (7, 5, 15))])
@pytest.mark.parametrize("turn", [False, True])
@pytest.mark.parametrize("dtype", [np.float32, np.int16])
def test_gathers(nin, nout, turn, dtype):
    rng = np.random.default_rng(11)
    whole = rng.integers(-1000, 2000, tuple(v + 1 for v in nin)).astype(dtype)
    labels = rng.integers(1, 6, whole.shape).astype(np.int8)
    box = tuple(slice(1, 1 + v) for v in nin)
    A = 9.0 * (R if turn else np.diag([1.0, 1.0, min(1.0, nin[2] / (9.0 * nout[2]))]))
    M = _map(A, nin, nout)
    ref, lref = oracle.warp(np.ascontiguousarray(whole[box]), M, nout,
                            lbl=np.ascontiguousarray(labels[box]), fill=-1000.0, label_fill=-3)
    out, lout = ctaug.warp_affine(torch.from_numpy(whole).cuda()[box], M,
                                  lbl=torch.from_numpy(labels).cuda()[box], fill=-1000.0,
                                  label_fill=-3, out_dim=nout)
    assert np.array_equal(lout.cpu().numpy(), lref)
    assert np.all(np.abs(out.cpu().numpy() - ref) <= 1e-5 * np.maximum(np.abs(ref), 1000.0))


@pytest.mark.parametrize("offset", [0.0, 3.0e6, -5.0e7])
def test_large_coordinates(offset):
    """Offsets past what the windows admit take the gathers; all is fill there."""
    rng = np.random.default_rng(6)
    img = rng.integers(-1000, 2000, (20, 22, 24)).astype(np.float32)
    M = _map(R, img.shape, (17, 18, 20))
    M[0, 3] += np.float32(offset)
    ref, _ = oracle.warp(img, M, (17, 18, 20), fill=5.0)
    out, _ = ctaug.warp_affine(torch.from_numpy(img).cuda(), M, fill=5.0, out_dim=(17, 18, 20))
    assert np.all(np.abs(out.cpu().numpy() - ref) <= 1e-5 * np.maximum(np.abs(ref), 1000.0))


def test_guard_keeps_nonfinite_voxels_out():
    """A sample exactly at -1 or n is fill, also beside infinite and NaN voxels."""
    n = (12, 10, 16)
    img = np.full(n, np.inf, dtype=np.float32)
    img[:, ::2] = np.nan
    for axis in range(3):
        M = np.concatenate([np.eye(3), np.zeros((3, 1))], axis=1).astype(np.float32)
        M[axis, 3] = -1.0              # output plane 0 of the axis lies at -1
        out, _ = ctaug.warp_affine(torch.from_numpy(img).cuda(), M, fill=2.5, out_dim=n)
        assert np.all(np.take(out.cpu().numpy(), 0, axis) == 2.5)
        M[axis, 3] = float(n[axis])
        out, _ = ctaug.warp_affine(torch.from_numpy(img).cuda(), M, fill=2.5, out_dim=n)
        assert np.all(out.cpu().numpy() == 2.5)


def test_nonfinite_displacements_give_fill():
    n = (11, 13, 18)
    rng = np.random.default_rng(7)
    img = rng.integers(-1000, 2000, n).astype(np.float32)
    lbl = rng.integers(1, 6, n).astype(np.int8)
    disp = rng.normal(0, 2, (3,) + n).astype(np.float32)
    bad = rng.random(n) < 0.1
    clean = disp.copy()
    disp[0][bad] = np.nan
    disp[1][bad & (rng.random(n) < 0.5)] = np.inf
    disp[2][rng.random(n) < 0.02] = -np.inf
    bad = ~np.isfinite(disp).all(0)
    M = np.concatenate([np.eye(3), np.zeros((3, 1))], axis=1).astype(np.float32)
    t = lambda a: torch.from_numpy(a).cuda()  # noqa: E731
    out, lout = ctaug.warp_displacement(t(img), M, t(disp), lbl=t(lbl), fill=3.5, label_fill=-2)
    ref, lref = ctaug.warp_displacement(t(img), M, t(clean), lbl=t(lbl), fill=3.5, label_fill=-2)
    out, lout, ref, lref = (x.cpu().numpy() for x in (out, lout, ref, lref))
    assert np.all(out[bad] == 3.5) and np.all(lout[bad] == -2)
    assert np.array_equal(out[~bad], ref[~bad]) and np.array_equal(lout[~bad], lref[~bad])

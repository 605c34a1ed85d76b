"""Non-finite entries of a field's gradient make every control of their voxel
non-finite, plane by plane and by passes, and leave the others as they are."""
import numpy as np
import pytest
import torch

import paper_1811_11226_amd as ctaug
from test_bspline_adjoint_route import _by_planes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,grid", [((9, 70, 40), (8, 8, 8)), ((9, 70, 200), (5, 6, 20)),
                                       ((16, 64, 401), (6, 64, 64)), ((6, 130, 1001), (7, 33, 16)),
                                       ((9, 70, 40), (5, 40, 30)), ((4, 300, 260), (9, 16, 16))])
def test_every_control_of_the_voxel(dims, grid):
    rng = np.random.default_rng(3)
    g = rng.normal(0, 1, (3,) + dims).astype(np.float32)
    clean = ctaug.bspline_upsample_adjoint(torch.from_numpy(g).cuda(), grid).cpu().numpy()
    at = [(0, 1, 3, 5), (1, dims[0] - 1, dims[1] - 4, dims[2] - 1), (2, 2, 30, 0)]
    for p, v in zip(at, (np.nan, np.inf, -np.inf)):
        g[p] = v
    out = ctaug.bspline_upsample_adjoint(torch.from_numpy(g).cuda(), grid).cpu().numpy()
    for comp, *p in at:
        touched = np.zeros(grid, dtype=bool)
        i = [min(int(np.floor(np.float32(v) * np.float32((G - 3) / (n - 1)))), G - 4)
             for v, n, G in zip(p, dims, grid)]
        touched[tuple(slice(a, a + 4) for a in i)] = True
        # a weight of 0 times the value is NaN, any other infinite or NaN
        assert not np.any(np.isfinite(out[comp][touched]))
        assert np.allclose(out[comp][~touched], clean[comp][~touched], rtol=1e-5, atol=1e-5)


def test_both_forms_are_meant():
    assert _by_planes((9, 70, 40), (8, 8, 8)) and _by_planes((16, 64, 401), (6, 64, 64))
    assert not _by_planes((9, 70, 40), (5, 40, 30)) and not _by_planes((4, 300, 260), (9, 16, 16))

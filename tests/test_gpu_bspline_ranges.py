"""The x sums of the control-grid adjoint on fields of many planes: a non-finite plane
reaches exactly the controls of its cell."""
import numpy as np
import pytest
import torch

import paper_1811_11226_amd as ctaug

pytestmark = pytest.mark.gpu


# Planes whose cell, by its own FP32 product, begins or ends a plane or two beside where
# x = (control - 1) h puts it; the last of the field; and plane numbers past 2^24.
@pytest.mark.parametrize("nx,gx,x", [(18276216, 41, 17314307), (18706216, 26, 17892899),
                                     (18816216, 21, 17770867), (18816216, 21, 18816215),
                                     (300001, 64, 299999), (117, 8, 58)])
def test_planes_reach_their_controls(nx, gx, x):
    grid = (gx, 4, 4)
    g = torch.zeros((3, nx, 1, 1), device="cuda")
    g[1, x] = float("nan")
    s = np.float32(x) * np.float32((gx - 3) / (nx - 1))
    first = int(min(np.floor(s), gx - 4))
    out = ctaug.bspline_upsample_adjoint(g, grid).cpu().numpy()
    touched = np.zeros((3,) + grid, dtype=bool)
    touched[1, first:first + 4] = True
    assert np.array_equal(np.isnan(out), touched)
    assert np.all(out[~touched] == 0.0)

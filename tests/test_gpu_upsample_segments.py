"""Upsampled fields whose rows are split over workgroups along z, bit for bit the
parity-mode field: ragged last segments, one and many rows, and a field past the number
of workgroups from which rows stay whole."""
import numpy as np
import pytest
import torch

import oracle
import paper_1811_11226_amd as ctaug

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,grid", [((1, 1, 257), (4, 4, 4)), ((1, 3, 5000), (4, 5, 64)),
                                       ((3, 17, 1537), (5, 6, 9)), ((40, 90, 513), (6, 7, 30)),
                                       ((70, 119, 515), (8, 8, 8)), ((130, 65, 300), (5, 4, 9))])
def test_segments(dims, grid):
    rng = np.random.default_rng(sum(dims))
    c = rng.normal(0, 4, (3,) + grid).astype(np.float32)
    u = ctaug.bspline_upsample(torch.from_numpy(c).cuda(), dims).cpu().numpy()
    assert np.array_equal(u, oracle.bspline_upsample_f32(c, dims))

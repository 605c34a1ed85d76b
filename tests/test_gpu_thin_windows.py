"""A plan's own reservation holds the whole window of a tile of inputs thinner than a
tile's footprint (the n + 4 cells that clamped coordinates reach), so that their tiles
are not split; and the plan's and single calls' bits agree there."""
import numpy as np
import pytest
import torch

import oracle
import paper_1811_11226_amd as ctaug
from test_gpu_fwd_windows import MAPS, _map

pytestmark = pytest.mark.gpu


def _pitch(e):
    p = (e + 3) & ~3
    return p if p & 4 else p + 4


def _window(M, nin, tile):
    e = [min(int(np.floor(np.abs(M[i, :3].astype(float)) @ (np.array(tile) - 1))) + 3, nin[i] + 4)
         for i in range(3)]            # without the rounding bound: at most the real one
    return e[0] * e[1] * _pitch(e[2])


@pytest.mark.parametrize("nin,nout,name", [((5, 5, 5), (16, 32, 16), "rotation"),
                                           ((8, 8, 8), (16, 16, 32), "rotation"),
                                           ((9, 8, 7), (40, 33, 37), "stretch"),
                                           ((40, 50, 1), (40, 50, 16), "worst"),
                                           ((1, 50, 40), (16, 50, 40), "worst"),
                                           ((2, 3, 2), (17, 18, 19), "reflected")])
def test_reservation_holds_the_window(nin, nout, name):
    rng = np.random.default_rng(8)
    img = rng.integers(-1000, 2000, nin).astype(np.float32)
    M = _map(MAPS[name], nin, nout)
    ti = torch.from_numpy(img).cuda()
    out = torch.empty(nout, device="cuda")
    plan = ctaug.BatchPlan([ctaug.make_job(ti, M, out, fill=-1000.0)], tile=(8, 16, 16))
    assert plan.tuning()[2] >= _window(M, nin, (8, 16, 16))
    plan.launch()
    one, _ = ctaug.warp_affine(ti, M, fill=-1000.0, out_dim=nout)
    torch.cuda.synchronize()
    assert torch.equal(out, one)
    plan.close()
    ref, _ = oracle.warp(img, M, nout, fill=-1000.0)
    assert np.all(np.abs(one.cpu().numpy() - ref) <= 1e-5 * np.maximum(np.abs(ref), 1000.0))

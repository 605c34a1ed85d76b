"""The autotune cache keeps a candidate that sizes its reservation from the jobs as one:
a plan of the same class with larger footprints reserves for its own, as a plan given
that tuning does, also through a saved cache."""
import numpy as np
import pytest
import torch

import paper_1811_11226_amd as ctaug

pytestmark = pytest.mark.gpu

NOUT = (24, 32, 32)


def _jobs(scale, keep):
    rng = np.random.default_rng(4)
    n = (40, 48, 48)
    ci, co = (np.array(n) - 1) / 2, (np.array(NOUT) - 1) / 2
    c, s = np.cos(0.4), np.sin(0.4)
    A = scale * np.array([[c, -s, 0], [s, c, 0], [0, 0, 1]])
    M = np.concatenate([A, (ci - A @ co)[:, None]], axis=1).astype(np.float32)
    jobs = []
    for _ in range(2):
        img = torch.from_numpy(rng.normal(0, 100, n).astype(np.float32)).cuda()
        out = torch.empty(NOUT, device="cuda")
        keep += [img, out]
        jobs.append(ctaug.make_job(img, M, out, fill=0.0))
    return jobs


def test_a_cached_choice_sizes_itself_from_each_plans_jobs(tmp_path):
    keep = []
    small, large = _jobs(0.2, keep), _jobs(1.1, keep)
    given = {}
    for name, jobs in (("small", small), ("large", large)):
        plan = ctaug.BatchPlan(jobs, tile=(8, 8, 32))
        given[name] = plan.tuning()
        plan.close()
    assert given["large"][2] > given["small"][2]
    ctaug.autotune_cache_clear()
    try:
        plan = ctaug.BatchPlan(small)
        best, _ = plan.autotune([((8, 8, 32), 0, 0, 0)], reps=1)
        assert best == plan.tuning() == given["small"]
        plan.close()
        for load in (False, True):
            if load:
                path = tmp_path / "cache.txt"
                ctaug.autotune_cache_save(path)
                ctaug.autotune_cache_clear()
                assert ctaug.autotune_cache_load(path) == 1
            for name, jobs in (("small", small), ("large", large)):
                assert ctaug.autotune_cache_lookup(jobs) == given[name]
                plan = ctaug.BatchPlan(jobs)
                assert plan.tuning() == given[name]
                plan.launch()
                torch.cuda.synchronize()
                plan.close()
    finally:
        ctaug.autotune_cache_clear()

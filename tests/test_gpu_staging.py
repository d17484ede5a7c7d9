"""Pinned host staging that solves keep from one to the next: the same results
from solves one after another, from two threads on streams of their own, and
with the staging freed in between."""
import threading

import numpy as np
import pytest

from tests.gpu_util import api, problem, to_dev, torch

pytestmark = pytest.mark.gpu


def test_solves_share_staging():
    a = api()
    made = []
    for name in ("c1", "c2_small"):
        p, vis = problem(name)
        made.append((a.pc_plan_create(p.uv, p.npix, p.fov_rad), to_dev(vis),
                     dict(alpha=p.alpha, delta=p.delta, max_iter=8)))
    a.pc_device_pool_trim(0)
    want = [a.pc_polyclean_solve(plan, v, **kw) for plan, v, kw in made]
    torch.cuda.synchronize()
    got = [[], []]
    errors = []

    def work(k):
        try:
            plan, v, kw = made[k]
            s = torch.cuda.Stream()
            with torch.cuda.stream(s):
                for turn in range(4):
                    got[k].append(a.pc_polyclean_solve(plan, v, **kw))
                    if turn == 1:
                        a.pc_device_pool_trim(0)
            s.synchronize()
        except Exception as e:  # noqa: BLE001
            errors.append(e)

    threads = [threading.Thread(target=work, args=(k,)) for k in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
    for w, rs in zip(want, got):
        for r in rs:
            assert r["objective"] == w["objective"] and np.array_equal(r["pix"], w["pix"])
    for plan, *_ in made:
        plan.close()

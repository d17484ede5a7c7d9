"""Work lists of the spread and the interpolation at the edges of their rules,
adjoint and forward against the exact sums: interpolation items of 256, 512 and
more visibilities and their remainders, spread items in one and in several
rounds of waves, and more plans than one readback launch takes."""
import numpy as np
import pytest

from oracle import operator
from tests.gpu_util import api, rel_l2, say, to_dev, torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,L", [(128, 255), (128, 256), (128, 257), (64, 40001), (64, 262144),
                                 (64, 262145), (128, 600001), (64, 3200001)])
def test_dense_patch(n, L):
    """At two dozen pixels (the exact sums take a second a million visibilities)."""
    a = api()
    rng = np.random.default_rng(L)
    fov = 0.02
    uv = rng.normal(0.0, 0.05, size=(L, 2)) / (fov / n)
    h = (rng.normal(size=L) + 1j * rng.normal(size=L)).astype(np.complex64)
    plan = a.pc_plan_create(uv, n, fov)
    img, mx, am = a.pc_adjoint_grid(plan, to_dev(h))
    img = img.cpu().numpy().reshape(-1)
    assert mx == np.abs(img).max() and am == int(np.abs(img).argmax())
    pix = np.unique(np.concatenate([[0, n - 1, n * n - 1, (n // 2) * n + n // 2, am],
                                    rng.choice(n * n, 19, replace=False)]))
    err = rel_l2(img[pix], operator.adjoint_pixels(uv, n, fov, h.astype(np.complex128), pix))
    x = np.zeros(n * n, np.float32)
    x[pix] = rng.normal(size=pix.size)
    out = a.pc_forward_grid(plan, to_dev(x.reshape(n, n))).cpu().numpy()
    ferr = rel_l2(out, operator.forward(uv, n, fov, pix, x[pix].astype(np.float64)))
    say("dense patch", n, L, "adjoint", err, "forward", ferr, plan.info)
    assert err <= 1e-4 and ferr <= 1e-4


def test_batch_of_many_plans():
    a = api()
    rng = np.random.default_rng(3)
    plans, vis = [], []
    for k in range(37):
        n = (16, 32, 64)[k % 3]
        L = 3 + 11 * k
        plans.append(a.pc_plan_create(rng.uniform(-0.4, 0.4, size=(L, 2)) / (0.02 / n), n, 0.02,
                                      nufft_eps=(1e-5, 1e-9)[k % 2]))
        vis.append(to_dev((rng.normal(size=L) + 1j * rng.normal(size=L)).astype(np.complex64)))
    imgs, mx, am = a.pc_adjoint_grid_batch(plans, vis)
    for p, v, img, m, i in zip(plans, vis, imgs, mx, am):
        want, wm, wi = a.pc_adjoint_grid(p, v)
        assert torch.equal(img, want) and (m, i) == (wm, wi)
    say("batch of", len(plans))

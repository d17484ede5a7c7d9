"""pc_adjoint_grid_batch of more requests than one readback launch takes (32),
with kernel widths of 8 and fewer and above 8 side by side: image and maximum
of each request equal the single call's bit for bit."""
import numpy as np
import pytest

from tests.gpu_util import api, to_dev, torch

pytestmark = pytest.mark.gpu


def test_forty_requests_of_several_widths():
    a = api()
    rng = np.random.default_rng(40)
    plans, vis = [], []
    for k in range(40):
        n = (64, 128, 256)[k % 3]
        fov = 0.02
        L = int(rng.integers(1, 3000))
        uv = rng.uniform(-0.45, 0.45, size=(L, 2)) / (fov / n)
        plans.append(a.pc_plan_create(uv, n, fov, nufft_eps=(1e-5, 1e-9, 1e-11, 1e-2)[k % 4]))
        vis.append(to_dev((rng.normal(size=L) + 1j * rng.normal(size=L)).astype(np.complex64)))
    alone = [a.pc_adjoint_grid(p, v) for p, v in zip(plans, vis)]
    alone = [(img.clone(), mx, am) for img, mx, am in alone]
    images, mx, am = a.pc_adjoint_grid_batch(plans, vis)
    torch.cuda.synchronize()
    for k, (img, m, i) in enumerate(alone):
        assert torch.equal(images[k], img), k
        assert mx[k] == m and am[k] == i, k
    for p in plans:
        p.close()

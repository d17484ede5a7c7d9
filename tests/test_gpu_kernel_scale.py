"""A constant factor on the FP32 gridding weights, which their random rounding
hides: the gridded forward of one unit pixel at the phase centre is one at every
(u, v), up to the kernel's aliasing, which averages out over random (u, v).

The mean's bound: the correction table's two rounded entries (6e-8 each at most),
the transform of a constant column and row (a few 1e-8 in the mean) and what is
left of the weights' own factor: 3e-7.
"""
import numpy as np
import pytest

from tests.gpu_util import api, say, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("W", range(5, 17))
def test_mean_of_the_forward_of_one_pixel(W):
    a = api()
    rng = np.random.default_rng(W)
    n, L = 64, 40000
    uv = rng.uniform(-0.49, 0.49, size=(L, 2)) / (0.02 / n)
    plan = a.pc_plan_create(uv, n, 0.02, nufft_eps=1.05 * 10.0 ** (1 - W))
    assert plan.info["kernel_width"] == W
    x = np.zeros((n, n), np.float32)
    x[n // 2, n // 2] = 1.0
    v = a.pc_forward_grid(plan, to_dev(x)).cpu().numpy().astype(np.complex128)
    say("W", W, "mean - 1", v.mean() - 1.0, "spread", np.std(v))
    assert abs(v.mean() - 1.0) <= 3e-7

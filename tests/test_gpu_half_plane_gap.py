"""Coverage that keeps away from v = 0 (a single baseline, a short snapshot, a
v-selected subset): the half plane's band then starts past zero frequency.
Adjoint, its maximum and the forward against the oracle's exact sums, the
batched and row-masked forms bit for bit against the single and full ones, and
the FP64 twin, on the LDS passes and on the register-held ones inside and
outside their window.  Tolerances as for the half plane's other edges.
"""
import numpy as np
import pytest

from oracle import operator
from tests.gpu_util import api, rel_l2, say, to_dev, torch
from tests.test_gpu_half_plane import _check

pytestmark = pytest.mark.gpu


def _turns(kind, n, rng):
    if kind == "one":
        return np.array([[0.1, 0.3]])
    if kind == "quarter":
        lo, hi = 0.25, 0.3
    elif kind == "edge":
        lo, hi = 0.45, 0.5
    else:  # fine cells 200 ... 400 from zero frequency
        lo, hi = 200 / (2.0 * n), 400 / (2.0 * n)
    t = np.stack([rng.uniform(-hi, hi, 301), rng.uniform(lo, hi, 301)], 1)
    t[1::2] *= -1.0
    return t


@pytest.mark.parametrize("n,kind", [(16, "one"), (128, "one"), (128, "quarter"), (128, "edge"),
                                    (512, "quarter"), (2048, "one"), (2048, "quarter"),
                                    (2048, "edge"), (4096, "cells"), (4096, "one"),
                                    (4096, "quarter"), (8192, "cells"), (8192, "one"),
                                    (8192, "quarter")])
def test_coverage_away_from_v_zero(n, kind):
    say("half plane without v = 0", n, kind)
    a = api()
    rng = np.random.default_rng(n)
    fov = 0.02
    turns = _turns(kind, n, rng)
    uv = turns / (fov / n)
    L = len(turns)
    h = (rng.normal(size=L) + 1j * rng.normal(size=L)).astype(np.complex64)
    plan = _check(uv, n, fov, h, samples=200)
    full = a.pc_adjoint_grid(plan, to_dev(h))[0]
    other = a.pc_plan_create(rng.uniform(-0.4, 0.4, size=(300, 2)) / (0.02 / 64), 64, 0.02)
    imgs, mx, _ = a.pc_adjoint_grid_batch([plan, other],
                                          [to_dev(h), to_dev(np.ones(300, np.complex64))])
    assert torch.equal(imgs[0], full) and mx[0] == float(full.abs().max())
    rows = [0, 5, n // 2, n - 1]
    mask = a.row_mask(n, rows)
    part = torch.zeros(n, n, device="cuda")
    a.pc_adjoint_grid_rows(plan, to_dev(h), mask, part)
    assert torch.equal(part[rows], full[rows])
    x = torch.zeros(n, n, device="cuda")
    x[rows] = torch.randn(4, n, device="cuda")
    assert torch.equal(a.pc_forward_grid_rows(plan, x, mask), a.pc_forward_grid(plan, x))
    if n <= 2048:
        plan = a.pc_plan_create(uv, n, fov, precision=a.PC_PREC_FP64)
        h = h.astype(np.complex128)
        img = a.pc_adjoint_grid_f64(plan, to_dev(h))[0].cpu().numpy().reshape(-1)
        pix = rng.choice(n * n, 200, replace=False)
        err = rel_l2(img[pix], operator.adjoint_pixels(uv, n, fov, h, pix))
        say("double", err)
        assert err <= 1e-4

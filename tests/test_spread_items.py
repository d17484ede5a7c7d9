"""The spread's work list on a band of few tiles: its items hold 64 visibilities
or more once there are tens of thousands, so that a plan's partial tiles stay a
fraction of its memory (items of 32 took 1.7 times the footprint)."""
import numpy as np
import pytest

from paper_2406_01342_amd import api


@pytest.mark.parametrize("n", [64, 128])
@pytest.mark.parametrize("L", [30001, 47051, 150001])
def test_partial_tiles_of_a_small_band(n, L):
    rng = np.random.default_rng(n)
    fov = 0.03
    r, th = 0.25 * np.sqrt(rng.random(L)), 2 * np.pi * rng.random(L)
    uv = np.stack([r * np.cos(th), r * np.sin(th)], 1) / (fov / n)
    M = 2 * n
    band = 8 * (M * (n + 32) + (n + 32) * n)   # half plane, pass-A buffer
    per_vis = L * (4 + 16 + 4 + 8 + 8)
    # each visibility reaches (1 + 5/32)^2 = 1.34 tiles; a partial tile is 8 KB
    # for at least 4 x 64 of them, one more per tile; lists under 128 KB
    partials = 8192 * (1.34 * L / 256 + (M // 32) ** 2)
    got = api.pc_plan_footprint(uv, n, fov)
    assert got <= 1.25 * (band + per_vis + partials) + (1 << 17)

"""Device memory of a non-coplanar plan: one w-plane's buffers beside the
per-visibility tables, whatever the number of planes (a group of planes works in
a workspace the plans of a device share)."""
import numpy as np
import pytest

from paper_2406_01342_amd import api


@pytest.mark.parametrize("n,fov,L,wmax", [(64, 0.06, 700, 9000.0), (1024, 0.07, 20001, 3700.0),
                                          (2048, 0.035, 5001, 20000.0)])
def test_footprint_counts_one_plane(n, fov, L, wmax):
    rng = np.random.default_rng(n)
    uv = rng.uniform(-0.49, 0.49, size=(L, 2)) / (fov / n)
    uv[:2] = [[0.4999 * n / fov, 0.4999 * n / fov], [-0.4999 * n / fov, -0.4999 * n / fov]]
    w = rng.uniform(-wmax, wmax, L)
    M = 2 * n
    plane = 8 * (M * M + M * n + L)           # grid, pass-A buffer, weighted visibilities
    tables = 1 << 20                          # tile and work lists
    per_vis = L * (4 + 16 + 4 + 8 + 8 + 8)
    # size classes are at most a quarter above the bytes asked for
    assert api.pc_plan_footprint(uv, n, fov, w=w) <= 1.25 * (plane + per_vis + tables) + 65536

"""The gridded operators at the edges of their forms, against the oracle's
exact sums: the half plane v >= 0 that coplanar plans grid (zero, negative and
half-turn v, coverage past the fine grid's edge, every kernel width), the
matrix-core spread's batches and items, the register-held passes at and past
the edge of their window, and the dictionary's point scale.

Tolerance: ten times the requested gridding accuracy, the operators' own
target (1e-4 for the default 1e-5), never below that 1e-4 in FP32 and 1e-8 in
FP64.  A kernel W cells wide needs each axis of the image raised by its
transform's fall, up to exp(0.62 W) at the edge and exp(0.14 W) half-way
there, and the rounding of the sums with it: FP32 is held at the inner half of
each axis when W > 8.
"""
import numpy as np
import pytest

from oracle import operator
from tests.gpu_util import api, rel_l2, say, to_dev, torch

pytestmark = pytest.mark.gpu


def _tol(eps):
    return max(10.0 * eps, 1e-4)


def _check(uv, n, fov, h, eps=1e-5, samples=400, seed=0):
    """Adjoint, its maximum, and the forward of a sparse image against the
    exact sums at sampled pixels (all of them on small images) and at every
    visibility."""
    a = api()
    rng = np.random.default_rng(seed)
    plan = a.pc_plan_create(uv, n, fov, nufft_eps=eps)
    img, mx, am = a.pc_adjoint_grid(plan, to_dev(h))
    got = img.cpu().numpy().astype(np.float64).reshape(-1)
    c = n // 2
    pix = np.arange(n * n) if n <= 64 else np.unique(np.concatenate(
        [[0, n - 1, n * n - 1, c * n + c, c * n, c, (c + 1) * n + c - 1, am],
         rng.choice(n * n, samples, replace=False)]))
    if eps < 0.9e-7:  # W > 8
        pix = pix[(abs(pix // n - c) < n // 4) & (abs(pix % n - c) < n // 4)]
    want = operator.adjoint_pixels(uv, n, fov, h.astype(np.complex128), pix)
    err = rel_l2(got[pix], want)
    say(n, len(uv), "eps", eps, "adjoint", err, plan.info)
    assert err <= _tol(eps)
    assert mx == np.abs(img.cpu().numpy()).max() and am == int(np.abs(got).argmax())
    val = rng.normal(size=pix.size)
    x = np.zeros(n * n, np.float32)
    x[pix] = val
    out = a.pc_forward_grid(plan, to_dev(x.reshape(n, n))).cpu().numpy()
    err = rel_l2(out, operator.forward(uv, n, fov, pix, x[pix].astype(np.float64)))
    say("forward", err)
    assert err <= _tol(eps)
    return plan


@pytest.mark.parametrize("n,eps", [(16, 1e-1), (16, 1e-5), (16, 1e-15), (32, 1e-7), (64, 1e-5),
                                   (64, 1e-12), (128, 1e-3), (1024, 1e-5)])
def test_half_plane_edges(n, eps):
    """v = 0, +-1/2 turn and their neighbours in FP64, v only negative, u on the
    same edges, coverage beyond one turn, and visibilities on tile edges."""
    rng = np.random.default_rng(n)
    fov = 0.02
    d = fov / n
    e = 1e-13
    edge = np.array([0.0, -0.0, e, -e, 0.5, -0.5, 0.5 - e, -0.5 + e, 0.5 + e, 0.25, -0.25])
    cells = np.arange(-n, n, max(1, n // 8)) / (2.0 * n)  # fine cells, tile edges among them
    pts = np.concatenate([edge, cells])
    uu, vv = np.meshgrid(pts, pts, indexing="ij")
    turns = np.concatenate([np.stack([uu.ravel(), vv.ravel()], 1),
                            rng.uniform(-1.3, 1.3, size=(257, 2)),
                            np.stack([rng.uniform(-0.5, 0.5, 65), -rng.uniform(0, 0.5, 65)], 1)])
    h = (rng.normal(size=len(turns)) + 1j * rng.normal(size=len(turns))).astype(np.complex64)
    _check(turns / d, n, fov, h, eps)
    a = api()
    plan = a.pc_plan_create(turns / d, n, fov, nufft_eps=eps, precision=a.PC_PREC_FP64)
    h = h.astype(np.complex128)
    img = a.pc_adjoint_grid_f64(plan, to_dev(h))[0].cpu().numpy().reshape(-1)
    pix = rng.choice(n * n, 200, replace=False)
    err = rel_l2(img[pix], operator.adjoint_pixels(turns / d, n, fov, h, pix))
    say("double", err)
    assert err <= max(10.0 * eps, 1e-8)


@pytest.mark.parametrize("L", [1, 31, 32, 33, 63, 97, 127, 128, 129, 513, 4097, 70001])
def test_spread_batches_and_items(L):
    """One dense patch of coverage: items of less than a batch, whole batches
    and their remainders, tiles shared by the waves of a workgroup and split
    into partial tiles, plus a few far visibilities in tiles of their own."""
    rng = np.random.default_rng(L)
    n, fov = 128, 0.02
    d = fov / n
    turns = rng.normal(0.0, 0.02, size=(L, 2))
    turns[: L // 50] = rng.uniform(-0.5, 0.5, size=(L // 50, 2))
    h = (rng.normal(size=L) + 1j * rng.normal(size=L)).astype(np.complex64)
    _check(turns / d, n, fov, h)


@pytest.mark.parametrize("n,reach", [(2048, 0.49), (4096, 2040), (4096, 2048 - 4), (4096, 2049),
                                     (4096, 2100), (8192, 2040), (8192, 2048 - 4), (8192, 2049),
                                     (8192, 2100)])
def test_register_passes_at_their_window(n, reach):
    """Coverage up to `reach` fine cells from zero frequency (turns when below
    one): inside the 4096-slot window, at its last cells, and just past it along
    one axis or both, where the full-length transforms take over; the batched
    adjoint and the row-masked pair equal the single and the full ones bit for
    bit on each path."""
    rng = np.random.default_rng(n + int(reach))
    fov = 0.05
    d = fov / n
    r = reach if reach < 1 else reach / (2.0 * n)
    for ru, rv in ((r, r), (r, 0.01), (0.01, r)):
        turns = rng.uniform(-1, 1, size=(501, 2)) * [ru, rv]
        turns[:4] = [[ru, rv], [-ru, -rv], [ru, -rv], [0.0, 0.0]]
        h = (rng.normal(size=501) + 1j * rng.normal(size=501)).astype(np.complex64)
        plan = _check(turns / d, n, fov, h, samples=200)
        a = api()
        full = a.pc_adjoint_grid(plan, to_dev(h))[0]
        other = a.pc_plan_create(rng.uniform(-0.4, 0.4, size=(300, 2)) / (0.02 / 64), 64, 0.02)
        h2 = np.ones(300, np.complex64)
        imgs, mx, am = a.pc_adjoint_grid_batch([plan, other], [to_dev(h), to_dev(h2)])
        assert torch.equal(imgs[0], full) and mx[0] == float(full.abs().max())
        mask = a.row_mask(n, [0, 5, n // 2, n - 1])
        part = torch.zeros(n, n, device="cuda")
        a.pc_adjoint_grid_rows(plan, to_dev(h), mask, part)
        rows = [0, 5, n // 2, n - 1]
        assert torch.equal(part[rows], full[rows]) and int((part != 0).any(1).sum()) <= 4
        x = torch.zeros(n, n, device="cuda")
        x[rows] = torch.randn(4, n, device="cuda")
        assert torch.equal(a.pc_forward_grid_rows(plan, x, mask), a.pc_forward_grid(plan, x))


@pytest.mark.parametrize("n", [128, 2048])
def test_maximum_of_zero_and_nan_images(n):
    """All pixels equal: index 0; a NaN visibility makes the image and its
    maximum NaN."""
    a = api()
    rng = np.random.default_rng(n)
    uv = rng.uniform(-0.4, 0.4, size=(100, 2)) / (0.02 / n)
    plan = a.pc_plan_create(uv, n, 0.02)
    h = torch.zeros(100, dtype=torch.complex64, device="cuda")
    assert a.pc_adjoint_grid(plan, h)[1:] == (0.0, 0)
    h[3] = complex("nan")
    img, mx, _ = a.pc_adjoint_grid(plan, h)
    assert bool(torch.isnan(img).all()) and np.isnan(mx)


@pytest.mark.parametrize("scales", [([0.0], [1.0]), ([0.0], [1.5]), ([2.0, 0.0, 5.0], [1.2, 1.0, 2.0]),
                                    ([0.0, 0.0], [1.0, 1.0])],
                         ids=["point", "scaled", "point-in-the-middle", "twice"])
def test_point_scale_is_the_image(scales):
    """A point scale of weight one is pc_adjoint_grid's image bit for bit,
    wherever it stands among the scales; maximum and lowest flat index over all
    scales as the images give them."""
    a = api()
    rng = np.random.default_rng(5)
    n = 256
    uv = rng.normal(0.0, 0.1, size=(3001, 2)) / (0.02 / n)
    h = to_dev((rng.normal(size=3001) + 1j * rng.normal(size=3001)).astype(np.complex64))
    plan = a.pc_plan_create(uv, n, 0.02)
    image = a.pc_adjoint_grid(plan, h)[0]
    out, mx, am = a.pc_adjoint_grid_ms(plan, h, *scales)
    for s, (sigma, gamma) in enumerate(zip(*scales)):
        if sigma == 0.0:
            assert torch.equal(out[s], image * gamma)
    flat = out.abs().reshape(-1)
    assert mx == float(flat.max()) and am == int((flat == flat.max()).nonzero()[0])


def test_w_planes_in_groups_of_any_size():
    """w ranges of one to many planes (groups of uneven sizes), against the
    exact sums."""
    a = api()
    rng = np.random.default_rng(8)
    n, fov, L = 64, 0.06, 700
    for wmax in (0.0, 300.0, 9000.0):
        uv = rng.uniform(-0.45, 0.45, size=(L, 2)) / (fov / n)
        w = np.full(L, 17.0) if wmax == 0.0 else rng.uniform(-wmax, wmax, L)
        h = (rng.normal(size=L) + 1j * rng.normal(size=L)).astype(np.complex64)
        plan = a.pc_plan_create(uv, n, fov, w=w)
        img = a.pc_adjoint_grid(plan, to_dev(h))[0].cpu().numpy()
        want = operator.adjoint(np.concatenate([uv, w[:, None]], 1), n, fov,
                                h.astype(np.complex128))
        say("w", wmax, plan.info, rel_l2(img, want))
        assert rel_l2(img, want) <= 1e-4

"""w-planes worked on together, in the workspace that the non-coplanar plans of a
device share: the same image bit for bit from several plans, threads and streams
as alone, under capture (plane by plane) and replayed; the memory given back;
and the w-stacked adjoint at fine grids 4096 and 8192 (register-held pass A
with several planes, inside and past its window) against the exact sums.
"""
import threading

import numpy as np
import pytest

from oracle import operator
from tests.gpu_util import api, say, to_dev, torch

pytestmark = pytest.mark.gpu


def _plan(n, L, seed, wmax, reach=0.45, fov=0.06, stream=None):
    rng = np.random.default_rng(seed)
    uv = rng.uniform(-reach, reach, size=(L, 2)) / (fov / n)
    w = rng.uniform(-wmax, wmax, L)
    h = to_dev((rng.normal(size=L) + 1j * rng.normal(size=L)).astype(np.complex64))
    return api().pc_plan_create(uv, n, fov, w=w), h, uv, w


def test_plans_threads_and_streams_share_it():
    """Plans of different sizes, each on a stream and thread of its own, many
    adjoints each without waiting in between."""
    a = api()
    made = [_plan(64, 700, 1, 9000.0), _plan(256, 5001, 2, 4000.0), _plan(512, 3001, 3, 2000.0)]
    alone = []
    for plan, h, *_ in made:
        alone.append(a.pc_adjoint_grid(plan, h)[0].clone())
    torch.cuda.synchronize()
    outs = [[] for _ in made]
    errors = []

    def work(k):
        try:
            plan, h = made[k][:2]
            s = torch.cuda.Stream()
            with torch.cuda.stream(s):
                for _ in range(8):
                    outs[k].append(a.pc_adjoint_grid(plan, h, want_max=False)[0])
            s.synchronize()
        except Exception as e:  # noqa: BLE001
            errors.append(e)

    threads = [threading.Thread(target=work, args=(k,)) for k in range(len(made))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors
    for k, got in enumerate(outs):
        for img in got:
            assert torch.equal(img, alone[k])


def test_capture_replays_and_memory_given_back():
    """A captured adjoint works plane by plane in the plan's own buffers: replays
    between eager adjoints of this and of another plan equal the eager image.
    With the last plan gone the workspace is parked, and a trim frees it."""
    a = api()
    a.pc_device_pool_trim(0)
    plan, h, *_ = _plan(256, 20001, 5, 4000.0)
    other, h2, *_ = _plan(128, 3001, 6, 4000.0)
    want = a.pc_adjoint_grid(plan, h)[0].clone()
    want2 = a.pc_adjoint_grid(other, h2)[0].clone()
    img = torch.empty_like(want)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        a.pc_adjoint_grid(plan, h, img, want_max=False)
    for _ in range(4):
        img.zero_()
        g.replay()
        assert torch.equal(a.pc_adjoint_grid(other, h2)[0], want2)
        assert torch.equal(a.pc_adjoint_grid(plan, h)[0], want)
        torch.cuda.synchronize()
        assert torch.equal(img, want)
    del g
    held = plan.info["footprint"] + other.info["footprint"]
    plan.close()
    other.close()
    released = a.pc_device_pool_trim(0)
    say("footprints", held, "released", released)
    assert released > held and released <= held + 2 * (512 << 20)
    assert a.pc_device_pool_trim(0) == 0


@pytest.mark.parametrize("n,reach", [(2048, 0.49), (4096, 0.2), (4096, 0.45)])
def test_w_adjoint_at_large_fine_grids(n, reach):
    plan, h, uv, w = _plan(n, 401, n, 3000.0, reach=reach)
    img, mx, am = api().pc_adjoint_grid(plan, h)
    img = img.cpu().numpy().reshape(-1)
    rng = np.random.default_rng(0)
    pix = np.unique(np.concatenate([rng.choice(n * n, 200, replace=False),
                                    [0, n - 1, n * n - 1, (n // 2) * n + n // 2, am]]))
    want = operator.adjoint_pixels(np.concatenate([uv, w[:, None]], 1), n, 0.06,
                                   h.cpu().numpy().astype(np.complex128), pix)
    err = np.max(np.abs(img[pix] - want)) / np.max(np.abs(want))
    say("w at", n, reach, plan.info, err)
    assert err <= 1e-4
    assert mx == np.abs(img).max() and am == int(np.abs(img).argmax())


def test_bytes_counted_for_the_rotating_pass():
    """Pass B of the w-planes reads each plane's pass-A buffer once, writes the
    image for the first plane and reads and writes it for every other."""
    a = api()
    n = 128
    plan, h, *_ = _plan(n, 3001, 4, 4000.0)
    info = plan.info
    a.pc_plan_profile(plan, True)
    a.pc_adjoint_grid(plan, h)
    stat = next(s for s in a.pc_plan_kernel_stats(plan) if s["name"] == "passB_adj_w")
    planes = info["w_planes"]
    assert planes > 8  # more than one group
    assert stat["bytes"] == planes * 8.0 * info["band_nv"] * n + 4.0 * n * n * (2 * planes - 1)


def test_last_use_followed_from_plan_to_plan():
    """Uses that end in an event and uses that the caller waited for (a maximum
    asked for), of plans on streams of their own, one of them destroyed right
    after its use: each image equals the one computed alone."""
    a = api()
    made = [_plan(64, 701, 11, 9000.0), _plan(256, 20001, 12, 4000.0), _plan(128, 3001, 13, 4000.0)]
    alone = [a.pc_adjoint_grid(plan, h)[0].clone() for plan, h, *_ in made]
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in made]
    outs = []
    for turn in range(6):
        for k, (plan, h, *_) in enumerate(made):
            with torch.cuda.stream(streams[k]):
                outs.append((k, a.pc_adjoint_grid(plan, h, want_max=(turn + k) % 3 == 0)[0]))
        if turn == 2:  # the plan that used the memory last
            made.pop()[0].close()
    for s in streams:
        s.synchronize()
    for k, img in outs:
        assert torch.equal(img, alone[k])
    for plan, *_ in made:
        plan.close()

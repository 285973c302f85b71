"""Going from scene to scene on one context: views' arrays, solver state and recorded
sequences are taken over where they fit.  Every result equals that of a context made for the
scene alone, over sizes that grow and shrink, more and fewer views, other references and
parameters between, rows with padding, images in device memory and a stream other than the
one before; a refused scene leaves the old one as it was."""
import ctypes as C

import numpy as np
import pytest

import scenegen as sg

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2104_06165_amd as pm  # noqa: E402


def scene(seed, W, H, n_src):
    return sg.make_scene(seed, sg.tiny_config(W, H, n_src=n_src, n_planes=3, n_textureless=1), device="cuda")


def run(ctx, n_src, lanes=0, iters=2, window=9):
    r = ctx.patchmatch(0, list(range(1, n_src + 1)), window, 1, iters, pm.Params(top_k=2, lanes=lanes))
    torch.cuda.synchronize()
    return [t.clone() for t in r]


def alone(s, *a, **k):
    ctx = pm.Context(0)
    try:
        ctx.set_scene(s)
        return run(ctx, len(s.images) - 1, *a, **k)
    finally:
        ctx.close()


def same(a, b):
    return all(torch.equal(x, y) for x, y in zip(a, b))


def test_scenes_in_turn():
    scenes = [scene(1, 96, 72, 3), scene(2, 96, 72, 3), scene(3, 130, 61, 5), scene(4, 40, 200, 2), scene(5, 96, 72, 4),
              scene(1, 96, 72, 3)]
    ref = [alone(s) for s in scenes]
    ctx = pm.Context(0)
    try:
        for order in (range(len(scenes)), reversed(range(len(scenes)))):
            for i in order:
                ctx.set_scene(scenes[i])
                n = len(scenes[i].images) - 1
                assert same(run(ctx, n), ref[i]), i
                assert same(run(ctx, n), ref[i]), i  # replayed
    finally:
        ctx.close()


def test_problems_between():
    """Other references, windows, iterations and lanes between, on the same and on the next
    scene: a recorded sequence serves only the launches it holds."""
    a, b = scene(6, 90, 64, 3), scene(7, 90, 64, 3)
    want = {}
    for k, s in enumerate((a, b)):
        for lanes in (0, 8):
            for it, win in ((2, 9), (1, 9), (2, 13)):
                want[k, lanes, it, win] = alone(s, lanes, it, win)
    ctx = pm.Context(0)
    try:
        for rep in range(2):
            for k, s in enumerate((a, b)):
                ctx.set_scene(s)
                for lanes in (0, 8):
                    for it, win in ((2, 9), (1, 9), (2, 13)):
                        assert same(run(ctx, 3, lanes, it, win), want[k, lanes, it, win])
                ctx.patchmatch(1, [0, 2], 7, 1, 1, pm.Params())
                ctx.patchmatch_batch([dict(ref=0, srcs=[1, 2], window=7, dilation=1)], 1)
    finally:
        ctx.close()


def test_streams():
    """Scenes and depth maps on different streams without the caller waiting between."""
    a, b = scene(8, 200, 150, 3), scene(9, 200, 150, 3)
    ra, rb = alone(a, iters=4), alone(b, iters=4)
    ctx = pm.Context(0)
    s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    p = pm.Params(top_k=2)
    try:
        for _ in range(3):
            with torch.cuda.stream(s1):
                ctx.set_scene(a)
                oa = ctx.patchmatch(0, [1, 2, 3], 9, 1, 4, p)
            with torch.cuda.stream(s2):
                ctx.set_scene(b)
                ob = ctx.patchmatch(0, [1, 2, 3], 9, 1, 4, p)
            torch.cuda.synchronize()
            assert same(oa, ra) and same(ob, rb)
    finally:
        ctx.close()


@pytest.mark.parametrize("pad", [0, 1, 13, 500])
@pytest.mark.parametrize("device", [False, True])
def test_rows_with_padding(pad, device):
    s = scene(10, 101, 67, 3)
    ref = alone(s)
    n = len(s.images)
    ims = (pm._Image * n)()
    keep = []
    for i, im in enumerate(s.images):
        H, W = im.shape
        buf = np.full((H, W + pad), 77, np.uint8)
        buf[:, :W] = im
        flat = buf.reshape(-1)[:(H - 1) * (W + pad) + W].copy()  # nothing behind the last pixel
        t = torch.from_numpy(flat)
        t = t.cuda() if device else t
        keep.append(t)
        ims[i] = pm._Image(W, H, W + pad if pad else 0, 0, t.data_ptr(), 1 if device else 0)
    dp = C.POINTER(C.c_double)
    arr = [np.ascontiguousarray(x, np.float64) for x in (s.K, s.R, s.t, np.tile(s.depth_range, (n, 1)))]
    ctx = pm.Context(0)
    try:
        ctx.set_scene(scene(11, 101, 67, 3))  # arrays to take over
        torch.cuda.synchronize()
        ctx._check(pm.lib().phimvs_set_views(ctx.h, n, ims, *[a.ctypes.data_as(dp) for a in arr]))
        assert same(run(ctx, 3), ref)
    finally:
        ctx.close()


def test_a_refused_scene_leaves_the_old_one():
    s = scene(12, 80, 60, 3)
    ref = alone(s)
    ctx = pm.Context(0)
    try:
        ctx.set_scene(s)
        bad = np.tile(np.eye(3), (4, 1, 1))
        bad[2, 0, 0] = np.nan
        with pytest.raises(pm.PhimvsError):
            ctx.set_views(s.images, bad, s.R, s.t, np.tile(s.depth_range, (4, 1)))
        assert same(run(ctx, 3), ref)
    finally:
        ctx.close()

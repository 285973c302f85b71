"""The consistency filter decides by a shorter arithmetic wherever that is certain and by the
written-out one elsewhere.  Maps that sit on the boundaries (whole- and half-pixel positions,
depth ratios, angles and re-projections at their thresholds, scenes far from the world's
origin, values that are no numbers, images of one row or column) and every number of
neighbours, against the FP64 oracle: every decision the same."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2104_06165_amd as pm  # noqa: E402


def run(K, R, t, depths, normals, par=None, ref=0):
    par = par or pm.FilterParams()
    n = len(depths)
    ctx = pm.Context(0)
    try:
        ctx.set_views([np.zeros(d.shape, np.uint8) for d in depths], K, R, t, np.tile([0.5, 50.0], (n, 1)))
        maps = [(i, torch.from_numpy(d).cuda(), torch.from_numpy(m).cuda()) for i, (d, m) in enumerate(zip(depths, normals))]
        nbrs = [i for i in range(n) if i != ref]
        g = [x.cpu().numpy() for x in ctx.filter(maps, ref, nbrs, par)]
    finally:
        ctx.close()
    o = oracle.consistency(dict(enumerate(depths)), dict(enumerate(normals)), K, R, t, ref, nbrs, par.max_rel_depth,
                           par.max_angle_deg, par.max_reproj_px, par.min_consistent)
    for a, b in zip(g, o):
        assert np.array_equal(a, b, equal_nan=a.dtype.kind == "f")
    return g[2]


def cams(n, f, c, t=None):
    K = np.array([[f, 0, c[0]], [0, f, c[1]], [0, 0, 1.0]])
    return (np.tile(K, (n, 1, 1)), np.tile(np.eye(3), (n, 1, 1)),
            np.zeros((n, 3)) if t is None else np.asarray(t, np.float64))


def maps(rng, n, H, W, spread=0.01, tilt=0.2, empty=0.05):
    d = [(4.0 * (1 + spread * rng.standard_normal((H, W)))).astype(np.float32) for _ in range(n)]
    m = [np.dstack([tilt * rng.standard_normal((H, W)), tilt * rng.standard_normal((H, W)), -np.ones((H, W))])
         for _ in range(n)]
    for x in d:
        x[rng.random((H, W)) < empty] = 0.0
    return d, [(v / np.linalg.norm(v, axis=-1, keepdims=True)).astype(np.float32) for v in m]


@pytest.mark.parametrize("shift", [0.0, 0.5, 1.0, 2.5])
def test_positions_on_whole_and_half_pixels(shift):
    rng = np.random.default_rng(int(10 * shift))
    K, R, t = cams(3, 64.0, (20.0, 11.0), t=[[0, 0, 0], [shift * 4 / 64, 0, 0], [0, shift * 4 / 64, 0]])
    d, m = maps(rng, 3, 23, 41)
    run(K, R, t, [np.full((23, 41), 4.0, np.float32)] * 3, m)
    assert run(K, R, t, d, m).max() > 0


def test_quantities_at_their_thresholds():
    # identical cameras, so that each test's quantity is known: depth ratio, normal angle
    K, R, t = cams(4, 64.0, (0.0, 0.0))
    H, W = 3, 64
    flat = np.tile(np.array([0, 0, -1], np.float32), (H, W, 1))
    lo = np.float32(4.0 / 1.015625)
    d = [np.full((H, W), v, np.float32) for v in (4.0, lo, np.nextafter(lo, np.float32(0)), np.nextafter(lo, np.float32(9)))]
    run(K, R, t, d, [flat] * 4, pm.FilterParams(max_rel_depth=0.015625))
    d = [np.full((H, W), 4.0, np.float32)] * 4
    n = []
    for a in (0.0, 60.0, np.nextafter(60.0, 0.0), 60.00001):
        v = np.tile(np.array([np.sin(np.radians(a)), 0, -np.cos(np.radians(a))], np.float32), (H, W, 1))
        n.append(v)
    run(K, R, t, d, n, pm.FilterParams(max_angle_deg=60.0))
    # a rectified pair: depth z and z (1 + e) re-project f b (1/z - 1/z') apart
    K, R, t = cams(2, 64.0, (31.5, 1.0), t=[[0, 0, 0], [-0.25, 0, 0]])
    z2 = np.float32(4.0 * 16 / 15.5)
    for px in (64 * 0.25 * (1 / 4.0 - 1 / float(z2)), 0.125, 0.12499999):
        run(K, R, t, [np.full((H, W), 4.0, np.float32), np.full((H, W), z2, np.float32)], [flat] * 2,
            pm.FilterParams(max_rel_depth=0.5, max_reproj_px=px, min_consistent=1))


@pytest.mark.parametrize("far", [0.0, 1e3, 1e7])
@pytest.mark.parametrize("tau", [0.3, 1.0, 50.0])
def test_scenes_away_from_the_origin(far, tau):
    rng = np.random.default_rng(5)
    Q = np.linalg.qr(rng.standard_normal((3, 3)))[0]
    Q, q = Q * np.sign(np.linalg.det(Q)), far * rng.standard_normal(3)
    K, R, t = cams(6, 90.0, (31.0, 17.5))
    K[1:3, 0, 1], K[1:3, 1, 1] = 2.0, 80.0  # skew, pixels that are not square
    for i in range(6):
        a = 0.05 * (i - 2)
        Ri = np.array([[np.cos(a), 0, -np.sin(a)], [0, 1, 0], [np.sin(a), 0, np.cos(a)]])
        R[i], t[i] = Ri @ Q.T, np.array([0.1 * (i - 2), 0.02 * i, 0.0]) - Ri @ (Q.T @ q)
    d, m = maps(rng, 6, 36, 63, tilt=0.3)
    run(K, R, t, d, m, pm.FilterParams(max_reproj_px=tau), ref=2)


@pytest.mark.parametrize("n", [1, 2, 3, 13])
def test_numbers_of_neighbours(n):
    rng = np.random.default_rng(n)
    K, R, t = cams(max(n, 2), 50.0, (15.0, 8.0), t=0.01 * rng.standard_normal((max(n, 2), 3)))
    d, m = maps(rng, max(n, 2), 17, 31)
    if n == 1:  # no neighbours: every pixel's count is 0
        ctx = pm.Context(0)
        try:
            ctx.set_views([np.zeros((17, 31), np.uint8)] * 2, K, R, t, np.tile([0.5, 50.0], (2, 1)))
            g = ctx.filter([(0, torch.from_numpy(d[0]).cuda(), torch.from_numpy(m[0]).cuda())], 0, [])
            assert int(g[2].max()) == 0 and float(g[0].abs().max()) == 0.0
        finally:
            ctx.close()
        return
    run(K, R, t, d, m)


@pytest.mark.parametrize("H,W", [(1, 1), (1, 40), (40, 1), (2, 2), (5, 300)])
def test_small_images(H, W):
    rng = np.random.default_rng(H * 1000 + W)
    K, R, t = cams(3, 50.0, ((W - 1) / 2, (H - 1) / 2), t=0.002 * rng.standard_normal((3, 3)))
    d, m = maps(rng, 3, H, W)
    run(K, R, t, d, m)
    K, R, t = cams(3, 50.0, ((W - 1) / 2, (H - 1) / 2))
    run(K, R, t, d, m)


def test_values_that_are_no_numbers():
    rng = np.random.default_rng(11)
    K, R, t = cams(3, 50.0, (15.0, 8.0), t=0.01 * rng.standard_normal((3, 3)))
    d, m = maps(rng, 3, 17, 31)
    for x in d:
        for v in (-1.0, np.nan, np.inf, 1e-30, 1e30):
            x[rng.random(x.shape) < 0.03] = v
    for x in m:
        for v in (np.nan, np.inf, -np.inf, 1e30):
            x[rng.random(x.shape) < 0.02] = v
    run(K, R, t, d, m)


@pytest.mark.parametrize("how,far", [("f32", 1e3), (6, 1e3), (4, 0.0), (4, 1e2), ("scaled", 1e3)])
def test_rotations_that_are_not_exact(how, far):
    """The short form is a reordering of the written-out one for any R, orthonormal or not."""
    rng = np.random.default_rng(18)
    K, R, t = cams(4, 280.0, (79.5, 59.5))
    while True:
        Q = np.linalg.qr(rng.standard_normal((3, 3)))[0]
        Q, q = Q * np.sign(np.linalg.det(Q)), far * rng.standard_normal(3)
        for i in range(4):
            a = 0.05 * (i - 1)
            Ri = np.array([[np.cos(a), 0, -np.sin(a)], [0, 1, 0], [np.sin(a), 0, np.cos(a)]]) @ Q.T
            R[i] = Ri.astype(np.float32) if how == "f32" else (Ri * (1 + 2.4e-5 * (i - 1)) if how == "scaled" else Ri.round(how))
            t[i] = np.array([0.1 * (i - 1), 0.02 * i, 0.0]) - Ri @ q
        if max(np.abs(r.T @ r - np.eye(3)).max() for r in R) < 0.99e-4:
            break
    d, m = maps(rng, 4, 120, 160, tilt=0.3)
    run(K, R, t, d, m, ref=1)

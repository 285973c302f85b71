"""The hypothesis selection's graph model on the GPU: bands of 32 rows walked by one wave each,
chunks of 16 columns between them.  Against the oracle's plain sequential decoder, bitwise, at
the edges of bands and chunks and on both sides of the rule that leaves small graphs to the
host (nodes >= 20 steps); refusals and infinite potentials as with the host's decoder."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2104_06165_amd as pm  # noqa: E402


@pytest.fixture(scope="module")
def ctx():
    c = pm.Context(0)
    yield c
    c.close()


def maps(W, H, kind, seed):
    """depth (H, W), hyp and cost (4, H, W): continuous values, or few values (ties)."""
    r = np.random.default_rng(seed)
    few = kind == "few"
    value = (lambda s: r.integers(4, 8, s)) if few else (lambda s: r.uniform(2, 6, s))
    d = np.where(r.uniform(size=(H, W)) < 0.4, value((H, W)), 0.0).astype(np.float32)
    h = np.where(r.uniform(size=(4, H, W)) < 0.75, value((4, H, W)), 0.0).astype(np.float32)
    c = (0.5 * r.integers(0, 4, h.shape) if few else r.uniform(0, 2, h.shape)).astype(np.float32)
    d[: H // 8, : W // 8] = 0
    h[:, : H // 8, : W // 8] = 0  # no states at all
    return d, h, c


def select(ctx, d, h, c, **kw):
    t = [torch.from_numpy(x).cuda() for x in (d, h, c)]
    return ctx.phi_select(*t, pm.PhiParams(**kw)).cpu().numpy()


# full size; the half-size graph is (W + 1) // 2 x (H + 1) // 2.  One band, one whole band, a row
# more; whole chunks of steps and one more or less; wide, tall, many bands; left to the host
SIZES = [(127, 61), (128, 64), (98, 66), (131, 65), (129, 128), (226, 194), (225, 191), (1601, 131), (160, 1279),
         (62, 66), (700, 12)]


@pytest.mark.parametrize("kind", ["any", "few"])
@pytest.mark.parametrize("W,H", SIZES)
def test_selection_is_the_oracles(ctx, W, H, kind):
    d, h, c = maps(W, H, kind, W + H)
    for it in (0, 1, 5):
        print(f"selection {W} x {H}, {kind}, {it} iterations", flush=True)
        g = select(ctx, d, h, c, iterations=it)
        o = oracle.phi_select(d, h.transpose(1, 2, 0), c.transpose(1, 2, 0), iterations=it)
        assert np.array_equal(g, o)


def test_refused_and_infinite_potentials(ctx):
    """A potential that is not positive refuses the call and leaves the output alone; an infinite
    potential or an infinite edge energy decodes as on the host."""
    W, H = 200, 192
    d, h, c = maps(W, H, "any", 3)
    free = np.argwhere((d[::2, ::2] <= 0) & (h[1, ::2, ::2] > 0))
    y, x = 2 * free[len(free) // 2]
    for cost in (2.5, np.nan):
        bad = c.copy()
        bad[1, y, x] = cost
        with pytest.raises(pm.PhimvsError):
            select(ctx, d, h, bad)
    t = [torch.from_numpy(a).cuda() for a in (d, h, bad)]
    out = torch.full((H, W), -7.0, device="cuda")
    p = pm._PhiParams(1.0, 0.1, 2.0, 8)
    rc = pm.lib().phimvs_phi_select(ctx.h, W, H, *[a.data_ptr() for a in t], pm.C.byref(p), out.data_ptr())
    assert rc != 0 and bool((out == -7.0).all())
    inf = c.copy()
    inf[1, y, x] = -np.inf
    for cost, k3 in ((inf, 2.0), (c, 1e200), (c, 1e100)):
        lab, dec = pm.phi_decode_host(d[::2, ::2].copy(), h[:, ::2, ::2].copy(), cost[:, ::2, ::2].copy(),
                                      pm.PhiParams(k3=k3))
        ref = dec[np.arange(H)[:, None] // 2, np.arange(W)[None, :] // 2].astype(np.float64)
        dist = np.where(h > 0, np.abs(h.astype(np.float64) - ref), np.inf)
        best = np.take_along_axis(h, dist.argmin(0)[None], 0)[0]
        want = np.where(d > 0, d, np.where((ref > 0) & np.isfinite(dist.min(0)), best, 0.0)).astype(np.float32)
        assert np.array_equal(select(ctx, d, h, cost, k3=k3), want)


def test_labels_that_tie_to_within_rounding(ctx):
    """Two states whose energies are equal but for the rounding of their logarithms (potentials in
    the ratio of 1 to 4 edges' potentials): the host's logarithms decide, whatever the size."""
    W = H = 256
    n2 = W // 2
    Y, X = np.mgrid[:n2, :n2]
    for seed in range(60):
        r = np.random.default_rng(seed)
        s = np.float32(r.uniform(0.5, 3))
        fixed = ((X + Y) % 2 == 0) & (r.random((n2, n2)) < 0.7)
        f = np.pad(fixed, 1).astype(int)
        m = f[:-2, 1:-1] + f[2:, 1:-1] + f[1:-1, :-2] + f[1:-1, 2:]
        free = ((X + Y) % 2 == 1) & (m > 0)
        # edges of (2 - 1/2)^2 and (2 - 1/4)^2 to each of m fixed nodes, potentials 49^m and 36^m
        k = 2.0 ** -np.ceil(np.log2(49.0**m)) * 2.0 ** -r.integers(0, 6, (n2, n2))
        d, h, c = np.zeros((H, W), np.float32), np.zeros((4, H, W), np.float32), np.zeros((4, H, W), np.float32)
        d[::2, ::2] = np.where(fixed, 4 * s, 0)
        for i, (v, base) in enumerate(((6 * s, 49.0), (5 * s, 36.0))):
            h[i, ::2, ::2] = np.where(free, v, 0)
            c[i, ::2, ::2] = 2 - base**m * k
        p = dict(k1=float(r.uniform(0.3, 3)), k2=1e-300, iterations=int(r.integers(0, 4)))
        _, dec = pm.phi_decode_host(d[::2, ::2].copy(), h[:, ::2, ::2].copy(), c[:, ::2, ::2].copy(), pm.PhiParams(**p))
        ref = dec[np.arange(H)[:, None] // 2, np.arange(W)[None, :] // 2].astype(np.float64)
        dist = np.where(h > 0, np.abs(h.astype(np.float64) - ref), np.inf)
        best = np.take_along_axis(h, dist.argmin(0)[None], 0)[0]
        want = np.where(d > 0, d, np.where((ref > 0) & np.isfinite(dist.min(0)), best, 0.0)).astype(np.float32)
        assert np.array_equal(select(ctx, d, h, c, **p), want), seed


@pytest.mark.parametrize("W,H,it", [(226, 194, 8), (401, 131, 3), (160, 300, 1), (130, 130, 0)])
def test_a_tie_among_other_nodes(ctx, W, H, it):
    """One pair of states that ties to within rounding, in a corner of a graph with up to four states a
    node: the whole graph is decoded with the host's logarithms."""
    for seed in range(3):
        d, h, c = maps(W, H, "any", 10 * W + seed)
        s = np.float32(np.random.default_rng(seed).uniform(0.5, 3))
        d[-14:, -14:], h[:, -14:, -14:] = 0, 0
        y, x = (H - 7) // 2 * 2, (W - 7) // 2 * 2  # a node and its left neighbour, alone
        d[y, x - 2] = 4 * s
        h[:2, y, x] = 6 * s, 5 * s
        c[:2, y, x] = 2 - 49 / 64, 2 - 36 / 64
        p = dict(k1=float(np.random.default_rng(seed).uniform(0.3, 3)), k2=1e-300, iterations=it)
        o = oracle.phi_select(d, h.transpose(1, 2, 0), c.transpose(1, 2, 0), **p)
        assert np.array_equal(select(ctx, d, h, c, **p), o)

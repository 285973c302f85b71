"""Split-lane launches at the edges of their plan: rows shorter than a workgroup's pixels, one
pixel more, many rows (fewer workgroups per row) and few, every number of lanes, so that pairs
get 4, 8 or 16 lanes for the same split of the sums.  Whole runs against the oracle in the
same order of the sums, as close as that allows (bitwise where the libraries' transcendental
functions agree), and the costs of hypotheses against those of planes."""
import numpy as np
import pytest

import oracle
import scenegen as sg

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2104_06165_amd as pm  # noqa: E402


def scene_of(W, H, n_src, seed=12):
    return sg.make_scene(seed, sg.tiny_config(W, H, n_src=n_src, n_planes=3, n_textureless=1), device="cuda")


@pytest.mark.parametrize("W,H,lanes,window,dilation", [
    (31, 24, 16, 5, 1), (32, 24, 8, 5, 1), (33, 24, 4, 7, 1), (40, 700, 16, 5, 2), (400, 20, 16, 9, 2), (97, 60, 2, 11, 1),
    (260, 80, 8, 11, 1), (64, 48, 16, 3, 1)])
def test_runs(W, H, lanes, window, dilation):
    scene = scene_of(W, H, 3)
    p = pm.Params(top_k=2, lanes=lanes)
    ctx = pm.Context(0)
    try:
        ctx.set_scene(scene)
        d, n, c = (t.cpu().numpy() for t in ctx.patchmatch(0, [1, 2, 3], window, dilation, 2, p))
    finally:
        ctx.close()
    pb = oracle.Problem.from_scene(scene, window, dilation, top_k=2, bilateral=True, sigma_s=(window - 1) / 2.0,
                                   seed=p.seed, lanes=lanes)
    od, on, oc = oracle.patchmatch(pb, 2)
    m = pb.valid_mask()
    assert ((c == oc) & (d == od))[m].mean() >= 0.999


def test_steps_without_the_librarys_initialisation():
    """The pixels' reference sums come from the initialisation's launches; a state the caller
    sets without one, and one after another problem's, starts without them."""
    scene = scene_of(90, 50, 3)
    for lanes in (0, 4, 16):
        res = []
        for init_first in (False, True):
            ctx = pm.Context(0)
            try:
                ctx.set_scene(scene)
                if init_first:
                    ctx.prepare(0, [1, 2, 3], 9, 1, pm.Params(top_k=2, lanes=lanes))
                    ctx.init_planes()
                    ctx.step(1, 0)
                    if init_first and lanes:
                        ctx.patchmatch(0, [1, 2], 13, 1, 1, pm.Params(lanes=lanes))  # another window's sums
                ctx.prepare(0, [1, 2, 3], 9, 1, pm.Params(top_k=2, lanes=lanes))
                g = torch.Generator().manual_seed(1)
                d = 3.0 + torch.rand((50, 90), generator=g)
                planes = torch.stack([0.1 * d, 0 * d, -torch.ones_like(d), d], -1).cuda()
                ctx.set_state(planes, torch.full((50, 90), 2.0, device="cuda"))
                ctx.step(1, 0)
                ctx.step(1, 1)
                res.append([t.clone() for t in ctx.get_state()])
            finally:
                ctx.close()
        assert torch.equal(res[0][0], res[1][0]) and torch.equal(res[0][1], res[1][1]), lanes


@pytest.mark.parametrize("lanes", [2, 4, 8, 16])
def test_hypothesis_costs(lanes):
    """phimvs_phi_costs scores hypothesis k as the fronto-parallel plane at its depth."""
    scene = scene_of(75, 50, 3)
    ctx = pm.Context(0)
    try:
        ctx.set_scene(scene)
        ctx.prepare(0, [1, 2, 3], 9, 1, pm.Params(top_k=2, lanes=lanes))
        g = torch.Generator().manual_seed(2)
        hyp = 2.0 + 4.0 * torch.rand((4, 50, 75), generator=g)
        hyp[torch.rand(hyp.shape, generator=g) < 0.4] = 0.0
        hyp = hyp.cuda()
        cost = ctx.phi_costs(hyp)
        for k in range(4):
            pl = torch.zeros((50, 75, 4), device="cuda")
            pl[..., 2] = -1.0
            pl[..., 3] = torch.where(hyp[k] > 0, hyp[k], torch.full_like(hyp[k], float("nan")))
            assert torch.equal(ctx.eval_cost(pl), cost[k])
        assert bool((cost[hyp <= 0] == pm.COST_MAX).all()) and bool((cost < pm.COST_MAX).any())
    finally:
        ctx.close()

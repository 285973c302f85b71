"""Propagation candidates by a wave per region (launches of up to 1024 blocks of 128 pixels)
against one thread per pixel (larger ones): maps estimated one by one and the same maps in one
batch that is large enough, bitwise, with each rule for leaving candidates out."""
import pytest

import scenegen as sg

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2104_06165_amd as pm  # noqa: E402


# compacted rows of exactly one and two waves of 64, one pixel more or less, several blocks of 128
@pytest.mark.parametrize("W,H", [(127, 131), (128, 130), (129, 130), (257, 121), (66, 260), (521, 133)])
@pytest.mark.parametrize("score_all", [0, 1, 2])
def test_one_by_one_and_in_a_batch(W, H, score_all):
    scene = sg.make_scene(W, sg.tiny_config(W, H, n_src=3, n_planes=3, n_textureless=1), device="cuda")
    per_map = ((W + 1) // 2 + 127) // 128 * H
    n = 1024 // per_map + 1
    assert per_map <= 1024 < n * per_map
    jobs = [dict(ref=i % 4, srcs=[v for v in range(4) if v != i % 4], window=(3, 5, 7)[i % 3], dilation=1,
                 params=pm.Params(top_k=2, score_all=score_all, seed=i)) for i in range(n)]
    print(f"{W} x {H}, score_all {score_all}: {n} maps", flush=True)
    ctx = pm.Context(0)
    try:
        ctx.set_scene(scene)
        batch = [[t.clone() for t in out] for out in ctx.patchmatch_batch(jobs, 3)]
        for j, b in zip(jobs, batch):
            one = ctx.patchmatch(j["ref"], j["srcs"], j["window"], j["dilation"], 3, j["params"])
            assert all(torch.equal(x, y) for x, y in zip(one, b))
    finally:
        ctx.close()

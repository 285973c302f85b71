"""The work-list order a context takes when no tuning was set: jobs whose sources' epipolar
lines cross many of their rows go by depth, others by pixel, also side by side in one
batch.  Each item's cost is computed on its own and the selection reads costs in slot
order, so every map equals the explicitly pixel-ordered one bit for bit."""
import pytest

import scenegen as sg

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2104_06165_amd as pm  # noqa: E402


@pytest.fixture(scope="module")
def grid():
    # 3 rows of 4 cameras; 6 x 8 degrees between neighbours: ~100 rows of vertical disparity
    return sg.make_multiview_scene(6, grid=(3, 4), refs_per_class=12, classes=[(417, 301, 11, 1)],
                                   n_src_range=(3, 3), master_size=(417, 301), n_planes=6)


def jobs(mv):
    """The camera at (1, 1) against its row (rows barely cross) and against its column, the
    column once more under the window-resize scheme."""
    return [dict(ref=5, srcs=[4, 6], window=11, dilation=1, params=pm.Params(top_k=2)),
            dict(ref=5, srcs=[1, 9], window=11, dilation=1, params=pm.Params(top_k=2)),
            dict(ref=9, srcs=[1, 5, 0], window=15, dilation=1, params=pm.Params(tap_radius=5))]


@pytest.mark.parametrize("use_graph", [False, True])
@pytest.mark.parametrize("pick", [[0], [1], [2], [0, 1], [0, 1, 2]])
def test_default_order_changes_no_result(grid, pick, use_graph):
    res = []
    for explicit in (True, False):
        ctx = pm.Context(0)
        try:
            ctx.set_views(grid.images, grid.K, grid.R, grid.t, grid.depth_ranges)
            if explicit:
                ctx.set_tuning(ctx.get_tuning())  # the same launch shape, pixel order asked for
            js = [jobs(grid)[i] for i in pick]
            out = ctx.patchmatch_batch(js, 3, use_graph=use_graph)
            if len(pick) == 1:
                j = js[0]
                one = ctx.patchmatch(j["ref"], j["srcs"], j["window"], j["dilation"], 3, j["params"])
                assert all(torch.equal(a, b) for a, b in zip(one, out[0]))
            res.append([t.clone() for o in out for t in o])
        finally:
            ctx.close()
    assert all(torch.equal(a, b) for a, b in zip(*res))


@pytest.mark.parametrize("pick", [[0], [1], [2], [0, 1, 2]])
def test_every_order_gives_the_same_maps(grid, pick):
    """The cameras' choice (a new context's tuning), pixel order, depth order and the cameras' choice
    with one kind of launch in depth order."""
    res = []
    ctx = pm.Context(0)
    try:
        ctx.set_views(grid.images, grid.K, grid.R, grid.t, grid.depth_ranges)
        t = ctx.get_tuning()
        assert t.order_by_depth == 8
        for order in (8, 0, 7, 9, 10, 12, 8):
            ctx.set_tuning(pm.Tuning(t.tile_rows, t.persistent, t.wgs_per_cu, order_by_depth=order))
            out = ctx.patchmatch_batch([jobs(grid)[i] for i in pick], 3)
            res.append([x.clone() for o in out for x in o])
    finally:
        ctx.close()
    assert all(torch.equal(a, b) for r in res[1:] for a, b in zip(res[0], r))

"""How the forward deals its regions to the waves: one region, fewer than one wave each, a few rounds by
stride, many rounds from the counters (8-pixel tiles of a large view, 16-pixel regions), ragged edges. The
visibility and the colours must not depend on it, and small ones are held against the oracle."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2603_27151_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("size", [(1, 1), (8, 8), (17, 9), (509, 333), (2701, 1733)])
def test_tiles_agree(size):
    from paper_2603_27151_amd import _lib, raster as R
    rng = np.random.Generator(np.random.PCG64(3))
    s = W.random_scene(rng, W.equilateral_soup(rng, W.uniform_ball(rng, 300), log_mean=-1.5), 4, 8, [8, 16, 4])
    ds = R.DeviceScene.from_host(s)
    v = W.View(size[0], size[1], 1, W.view_proj((0.0, 0.0, 3.0), size[0], size[1]))
    vs = R.Views.from_list([v])
    ctx = _lib.Ctx(torch.cuda.current_device())
    got = []
    for tile in (8, 16, 32):
        ctx.set_tile(tile)
        vis, col, _ = R.rasterize_fwd(ds, vs, R.Opts(seed=5), ctx=ctx)
        got.append((vis.cpu().numpy(), col.cpu().numpy()))
    for vis, col in got[1:]:
        assert np.array_equal(vis, got[0][0]) and np.array_equal(col, got[0][1])
    if size[0] <= 509:
        rvis, _, _, _ = O.forward(s, v, O.Opts(seed=5))
        assert np.array_equal(got[0][0].view(np.uint64).reshape(rvis.shape), rvis)

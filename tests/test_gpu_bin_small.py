"""Binning of calls too small for the histogram chunks: chunks of 16, 64 and 256 triangles with a ragged
last one, triangles of many tiles beside small and culled ones, views with and without spread counters
(up to 8,192, up to 16,384 and more tiles), scans by one workgroup and by three launches. The number of list
entries is the oracle's bounding boxes' by count, and the visibility is the oracle's."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2603_27151_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _boxes(verts, view, tile):
    """Tiles touched by the triangles' pixel boxes (float64; vertices chosen so that none is near a tie)."""
    v = np.concatenate([verts.astype(np.float64), np.ones(verts.shape[:2] + (1,))], 2) @ view.M.astype(np.float64).T
    X = np.rint(256 * (view.width / 2 * (v[..., 0] / v[..., 3] + 1)))
    Y = np.rint(256 * (view.height / 2 * (1 - v[..., 1] / v[..., 3])))
    n = 0
    for i in range(len(verts)):
        if (v[i, :, 3] < 0.1).any():
            continue
        x0, x1 = max((X[i].min() + 127) // 256, 0), min((X[i].max() - 128) // 256, view.width - 1)
        y0, y1 = max((Y[i].min() + 127) // 256, 0), min((Y[i].max() - 128) // 256, view.height - 1)
        if x0 <= x1 and y0 <= y1:
            n += int((x1 // tile - x0 // tile + 1) * (y1 // tile - y0 // tile + 1))
    return n


@pytest.mark.parametrize("T", [1, 17, 64, 300, 5003])
@pytest.mark.parametrize("size,tile", [((9, 5), 16), ((640, 361), 16), ((1024, 1040), 8), ((1301, 1033), 8)])
def test_small_chunks(T, size, tile):
    from paper_2603_27151_amd import _lib, raster as R
    rng = np.random.Generator(np.random.PCG64(T))
    verts = W.equilateral_soup(rng, W.uniform_ball(rng, T, 0.8), log_mean=-2.5)
    verts[::9] *= 3.0                       # some large, some behind the camera
    verts[::31, :, 2] += 4.0
    s = W.random_scene(rng, verts, 4, 8, [8, 16, 4])
    v = W.View(size[0], size[1], 2, W.view_proj((0.0, 0.0, 3.0), size[0], size[1]))
    ctx = _lib.Ctx(torch.cuda.current_device())
    ctx.set_tile(tile)
    vis, _, _ = R.rasterize_fwd(R.DeviceScene.from_host(s), R.Views.from_list([v]), R.Opts(seed=9), ctx=ctx)
    got = ctx.stats()["bin_entries"]
    want = _boxes(verts, v, tile)
    assert abs(got - want) <= 2e-3 * want + 1, (got, want)   # a box edge may round the other way in float64
    if size[0] < 1000:
        rvis, _, _, _ = O.forward(s, v, O.Opts(seed=9))
        assert np.array_equal(vis.cpu().numpy().view(np.uint64).reshape(rvis.shape), rvis)

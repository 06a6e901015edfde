"""The forward's search for a region's view, by the whole wave: one view, the edges of one view per
lane, two levels (65 views and more) and three (more than 4096). Views of the same size and camera
must show the same, whatever their place in the call (threshold mode: no random draws)."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2603_27151_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

SIZES = [(9, 7), (33, 20), (1, 1), (16, 16)]


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 130, 4096, 4097, 5000])
def test_views_agree(n):
    from paper_2603_27151_amd import raster as R
    rng = np.random.Generator(np.random.PCG64(5))
    s = W.random_scene(rng, W.equilateral_soup(rng, W.uniform_ball(rng, 20), log_mean=-0.7), 4, 8, [8, 16, 4])
    views = [W.View(w, h, i, W.view_proj((0.0, 0.0, 3.0), w, h)) for i in range(n) for w, h in [SIZES[(i * 7) % 4]]]
    vis, col, _ = R.rasterize_fwd(R.DeviceScene.from_host(s), R.Views.from_list(views), R.Opts(mode=1))
    vis, col = vis.cpu().numpy().view(np.uint64).ravel(), col.cpu().numpy().reshape(-1, 3)
    ref, at = {}, 0
    for v in views:
        size, m = (v.width, v.height), v.width * v.height
        got = vis[at:at + m], col[at:at + m]
        if size not in ref:
            assert np.array_equal(got[0].reshape(v.height, v.width), O.forward(s, v, O.Opts(mode=1))[0])
            ref[size] = got
        assert np.array_equal(got[0], ref[size][0]) and np.array_equal(got[1], ref[size][1])
        at += m

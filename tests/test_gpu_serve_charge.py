"""The serving loop's charge for small requests bounds what their renders allocate, for every decoder shape (the
decoder's parameters and the context's counters weigh most where the image is small)."""
import numpy as np
import pytest

from paper_2603_27151_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("tile", [8, 16, 32])
@pytest.mark.parametrize("dims", [[8, 16, 4], [16, 32, 32, 4], [32, 64, 64, 4]], ids=lambda d: "-".join(map(str, d)))
def test_small_requests(dims, tile):
    from paper_2603_27151_amd import raster as R
    from paper_2603_27151_amd import serve as SV
    for T in (10, 1000):
        rng = np.random.Generator(np.random.PCG64(1))
        soup = W.random_scene(rng, W.equilateral_soup(rng, W.uniform_ball(rng, T)), 4, dims[0], dims)
        srv = SV.Server([R.DeviceScene.from_host(soup)], tile=tile, n_streams=1, max_batch=1)
        for w, h in [(32, 32), (64, 64), (160, 90), (640, 360)]:
            v = W.View(w, h, 3, W.view_proj((0.4, 0.2, 3.0), w, h))
            assert srv.measure_request(0, v) <= srv.need(0, v), f"{T} triangles, {w} x {h}"

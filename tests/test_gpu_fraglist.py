"""The fragments a backward takes from the forward's log and those it finds again by a walk with the winners
known: the same gradients (up to the order of float32 sums), whatever part of the image carries colour
gradients and score weights, for every tile side, ragged views and log p from either."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2603_27151_amd import workloads as W
from tests import parity as PT

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _setup(T=400):
    rng = np.random.Generator(np.random.PCG64(21))
    s = W.random_scene(rng, W.equilateral_soup(rng, W.uniform_ball(rng, T), log_mean=-1.5), 8, 16, [16, 32, 32, 4])
    sizes = [(131, 77), (64, 64), (1, 9), (300, 41)]
    eyes = W.fibonacci_sphere(len(sizes), 3.0)
    return s, [W.View(w, h, i, W.view_proj(eyes[i], w, h)) for i, (w, h) in enumerate(sizes)]


@pytest.mark.parametrize("tile", [8, 16, 32])
@pytest.mark.parametrize("weights", ["all", "half", "none", "few colours"])
@pytest.mark.parametrize("edge_pairs", [0, 2])
def test_log_and_walk_agree(tile, weights, edge_pairs):
    from paper_2603_27151_amd import _lib, raster as R
    s, views = _setup()
    ds, vs = R.DeviceScene.from_host(s), R.Views.from_list(views)
    ctx = _lib.Ctx(torch.cuda.current_device())
    ctx.set_tile(tile)
    log, walk = (R.Opts(seed=3, reuse_bins=k, edge_pairs=edge_pairs) for k in (1, 0))
    vis, col, logp = R.rasterize_fwd(ds, vs, log, want_logp=True, ctx=ctx)
    gen = torch.Generator(device="cuda").manual_seed(1)
    gc = torch.randn(col.shape, device="cuda", generator=gen)
    gl = torch.rand(col.shape[0], device="cuda", generator=gen)
    if weights == "half":
        gl[::2] = 0
    if weights == "few colours":
        gl[:] = 0
        gc[torch.arange(len(gc), device="cuda") % 7 != 0] = 0
    gl = None if weights == "none" else gl
    a = R.rasterize_bwd(ds, vs, log, vis, col, gc, gl, ctx=ctx)
    b = R.rasterize_bwd(ds, vs, walk, vis, col, gc, gl, ctx=ctx)
    c = R.rasterize_bwd(ds, vs, log, vis, col, gc, gl, ctx=ctx)   # after the walk: no log of these bins any more
    for x in (b, c):
        PT.assert_grads([t.cpu().numpy() for t in x], [t.cpu().numpy() for t in a], tol=1e-5)
    # log p from the walk (no log kept) and from the log
    logp2 = R.rasterize_fwd(ds, vs, walk, want_logp=True, ctx=ctx)[2]
    ref = np.concatenate([O.forward(s, v, O.Opts(seed=3))[2].ravel() for v in views])
    for x in (logp, logp2):
        assert np.max(np.abs(x.cpu().numpy() - ref)) <= 1e-5 * max(1.0, np.abs(ref).max())

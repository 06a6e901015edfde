"""What an eager pass has to have sized for a static-mode one that follows it."""
import numpy as np
import pytest

from paper_2603_27151_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("dims", [[8, 16, 4], [16, 32, 32, 4], [32, 64, 64, 4]], ids=lambda d: "-".join(map(str, d)))
def test_forward_after_a_backward(dims):
    """A static-mode forward needs no more than its binning, which a backward makes too."""
    from paper_2603_27151_amd import _lib, raster as R
    rng = np.random.Generator(np.random.PCG64(4))
    s = W.random_scene(rng, W.equilateral_soup(rng, W.uniform_ball(rng, 200), log_mean=-1.0), 4, dims[0], dims)
    ds, vs = R.DeviceScene.from_host(s), R.Views.from_list([W.View(90, 70, 1, W.view_proj((0.0, 0.0, 3.0), 90, 70))])
    opts = R.Opts(seed=9)
    vis, col, _ = R.rasterize_fwd(ds, vs, opts, ctx=_lib.Ctx(torch.cuda.current_device()))
    ctx = _lib.Ctx(torch.cuda.current_device())
    R.rasterize_bwd(ds, vs, opts, vis, col, torch.ones_like(col), ctx=ctx)
    ctx.set_static(True)
    vis2, col2, _ = R.rasterize_fwd(ds, vs, opts, ctx=ctx)
    torch.cuda.synchronize()
    ctx.check_overflow()
    assert torch.equal(vis, vis2) and torch.equal(col, col2)
    ctx.close()

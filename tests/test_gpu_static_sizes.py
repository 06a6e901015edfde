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


def test_after_a_log_that_overflowed():
    """The first forward of a deep soup overflows its log, and the backward makes one of its own, of few entries. A
    static-mode repeat takes the forward's log, cut, and reports that; eager again, and then static, it fits."""
    from paper_2603_27151_amd import _lib, raster as R
    rng = np.random.Generator(np.random.PCG64(4))
    z = np.linspace(-0.5, 0.5, 40, dtype=np.float32)
    v = np.stack([np.stack([np.array(p, np.float32) for p in ((-9, -9, d), (9, -9, d), (0, 12, d))]) for d in z])
    s = W.random_scene(rng, v, 2, 8, [8, 16, 4])
    s.mlp[-1] = -6.0   # almost transparent: nearly every layer of a pixel is decoded
    n = 2048
    ds, vs = R.DeviceScene.from_host(s), R.Views.from_list([W.View(n, n, 1, W.view_proj((0.0, 0.0, 3.0), n, n))])
    ctx = _lib.Ctx(torch.cuda.current_device())
    gc = torch.zeros(n * n, 3, device="cuda")
    opts = R.Opts(seed=9, edge_pairs=2, reuse_bins=1)

    def step():
        vis, col, _ = R.rasterize_fwd(ds, vs, opts, ctx=ctx)
        return (vis, col) + R.rasterize_bwd(ds, vs, opts, vis, col, gc, ctx=ctx)

    plain, small = R.Opts(seed=9, edge_pairs=2), R.Views.from_list([W.View(64, 64, 1, W.view_proj((0.0, 0.0, 3.0), 64, 64))])
    vis, col, _ = R.rasterize_fwd(ds, small, plain, ctx=ctx)
    g0 = torch.zeros(64 * 64, 3, device="cuda")
    g0[torch.nonzero(vis != -1)[::500, 0]] = 1.0
    R.rasterize_bwd(ds, small, plain, vis, col, g0, ctx=ctx)   # few fragments: the backward's next log is small
    vis, _, _ = R.rasterize_fwd(ds, vs, plain, ctx=ctx)
    gc[torch.nonzero(vis != -1)[::50_000, 0]] = 1.0
    want = step()
    ctx.set_static(True)
    step()
    torch.cuda.synchronize()
    with pytest.raises(_lib.SoupError, match="overflowed"):
        ctx.check_overflow()
    ctx.set_static(False)
    for static in (False, True):
        ctx.set_static(static)
        got = step()
        torch.cuda.synchronize()
        ctx.check_overflow()
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
        for a, b in zip(got[2:], want[2:]):   # sums of floats in another order
            assert float((a - b).norm()) <= 1e-5 * float(b.norm())
    ctx.close()

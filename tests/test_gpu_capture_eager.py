"""Eager calls on a stream that captures are refused, before anything is enqueued or kept: a backward that finds
everything it needs from the last forward in place, and a forward, after which a static-mode call still finds the
descriptors on the device that it compares with. The capture itself goes on and ends."""
import numpy as np
import pytest

from paper_2603_27151_amd import workloads as W
from paper_2603_27151_amd import _lib

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

SIZE = (90, 70)
P = SIZE[0] * SIZE[1]


def _captured(fn):
    """What fn raises on a capturing stream."""
    side, err = torch.cuda.Stream(), None
    side.wait_stream(torch.cuda.current_stream())
    g = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        g.capture_begin()
        try:
            fn()
        except _lib.SoupError as e:
            err = e
        g.capture_end()
    return err


def _views(R, n=1):
    return R.Views.from_list([W.View(*SIZE, i, W.view_proj((0.3 * i, 0.0, 3.0), *SIZE)) for i in range(n)])


def _scene(R, rng):
    return R.DeviceScene.from_host(W.random_scene(
        rng, W.equilateral_soup(rng, W.uniform_ball(rng, 200), log_mean=-1.0), 4, 8, [8, 16, 4]))


def test_backward_from_the_log():
    from paper_2603_27151_amd import raster as R
    ds, vs = _scene(R, np.random.Generator(np.random.PCG64(4))), _views(R)
    ctx, opts = _lib.Ctx(torch.cuda.current_device()), R.Opts(seed=9, reuse_bins=1)
    gc, gl = torch.ones(P, 3, device="cuda"), torch.ones(P, device="cuda")
    vis, col, _ = R.rasterize_fwd(ds, vs, opts, ctx=ctx)
    want = R.rasterize_bwd(ds, vs, opts, vis, col, gc, gl, ctx=ctx)
    R.rasterize_fwd(ds, vs, opts, ctx=ctx, out=(vis, col, None))
    got = [torch.empty_like(t) for t in want]
    torch.cuda.synchronize()
    bwd = lambda: R.rasterize_bwd(ds, vs, opts, vis, col, gc, gl, ctx=ctx, out=got)
    err = _captured(bwd)
    assert err is not None and err.status == 4
    bwd()
    for a, b in zip(got, want):
        assert float((a - b).norm()) <= 1e-5 * float(b.norm())
    ctx.close()


@pytest.mark.parametrize("level", [3, 6])   # sorted; per pixel
def test_paper_backward_from_the_log(level):
    from paper_2603_27151_amd import raster as R
    rng = np.random.Generator(np.random.PCG64(4))
    T = 50
    verts = W.equilateral_soup(rng, W.uniform_ball(rng, T), log_mean=-1.0)
    ds = R.PDeviceScene(*(torch.from_numpy(a.astype(np.float32)).cuda() for a in (
        verts, rng.random((T, R.mc_vertices(level), 8)), rng.standard_normal(_lib.PMLP_PARAMS) * 0.3)), level)
    vs = _views(R)
    ctx, opts = _lib.Ctx(torch.cuda.current_device()), R.Opts(seed=9, reuse_bins=1)
    gc, gl = torch.ones(P, 3, device="cuda"), torch.ones(P, device="cuda")
    vis, col, _ = R.pforward(ds, vs, opts, ctx=ctx)
    want = R.pbackward(ds, vs, opts, vis, col, gc, gl, ctx=ctx)
    R.pforward(ds, vs, opts, ctx=ctx, out=(vis, col, None))
    got = [torch.empty_like(t) for t in want]
    torch.cuda.synchronize()
    bwd = lambda: R.pbackward(ds, vs, opts, vis, col, gc, gl, ctx=ctx, out=got)
    err = _captured(bwd)
    assert err is not None and err.status == 4
    bwd()
    for a, b in zip(got, want):
        assert float((a - b).norm()) <= 1e-5 * float(b.norm())
    ctx.close()


def test_forward_leaves_the_descriptors():
    from paper_2603_27151_amd import raster as R
    ds, two, one = _scene(R, np.random.Generator(np.random.PCG64(4))), _views(R, 2), _views(R, 1)
    ctx, opts = _lib.Ctx(torch.cuda.current_device()), R.Opts(seed=9)
    out = (torch.empty(2 * P, dtype=torch.int64, device="cuda"), torch.empty(2 * P, 3, device="cuda"), None)
    R.rasterize_fwd(ds, two, opts, ctx=ctx, out=out)
    want = out[1].clone()
    torch.cuda.synchronize()
    err = _captured(lambda: R.rasterize_fwd(ds, one, opts, ctx=ctx, out=out))
    assert err is not None and err.status == 4
    ctx.set_static(True)
    with pytest.raises(_lib.SoupError, match="previous call"):   # not the views on the device
        R.rasterize_fwd(ds, one, opts, ctx=ctx, out=out)
    R.rasterize_fwd(ds, two, opts, ctx=ctx, out=out)
    torch.cuda.synchronize()
    ctx.check_overflow()
    assert torch.equal(out[1], want)
    ctx.close()

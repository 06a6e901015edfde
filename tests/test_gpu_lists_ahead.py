"""Tile lists scattered and sorted ahead, into a buffer that an earlier call sized and that proves too small: they
are made again, for small chunks (pairs dealt to a workgroup), large ones counted in the LDS, and large ones of a
view with more tiles than that holds. A context whose first call it is makes them once: the same results."""
import numpy as np
import pytest

from paper_2603_27151_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("T,n,size,log_mean", [(300, 2, (200, 150), -2.0), (60, 520, (40, 36), -2.0),
                                               (1_050_000, 1, (1500, 1400), -6.0)], ids=["small", "lds", "global"])
def test_made_again(T, n, size, log_mean):
    from paper_2603_27151_amd import _lib, raster as R
    rng = np.random.Generator(np.random.PCG64(6))
    s = W.random_scene(rng, W.equilateral_soup(rng, W.uniform_ball(rng, T), log_mean=log_mean), 2, 8, [8, 16, 4])
    ds = R.DeviceScene.from_host(s)
    vs = R.Views.from_list([W.View(*size, i, W.view_proj((0.0, 0.1, 3.0), *size)) for i in range(n)])
    opts = R.Opts(seed=2)
    centre = ds.verts.mean(dim=1, keepdim=True)
    big = R.DeviceScene((centre + 4.0 * (ds.verts - centre)).contiguous(), ds.feats, ds.mlp, ds.dims)
    ctx, fresh = (_lib.Ctx(torch.cuda.current_device()) for _ in range(2))
    R.rasterize_fwd(ds, vs, opts, ctx=ctx)
    small_lists = ctx.stats()["bin_entries"]
    got = R.rasterize_fwd(big, vs, opts, want_logp=True, ctx=ctx)
    want = R.rasterize_fwd(big, vs, opts, want_logp=True, ctx=fresh)
    assert ctx.stats()["bin_entries"] > 1.25 * small_lists   # past the buffer's headroom
    assert ctx.stats()["bin_entries"] == fresh.stats()["bin_entries"]
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
    assert float((got[2] - want[2]).norm()) <= 1e-5 * float(want[2].norm())   # log p: sums in another order
    ctx.close()
    fresh.close()

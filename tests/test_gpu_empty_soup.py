"""Forward and backward of an empty soup that has no parameters at all (every scene pointer NULL, as the
interface allows for T = 0): background, and zero gradients of the decoder, added to or overwritten."""
import ctypes as C

import numpy as np
import pytest

from paper_2603_27151_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

VIEWS = [W.View(w, h, 1, W.view_proj((0.0, 0.0, 3.0), w, h)) for w, h in [(33, 20), (8, 8)]]
P = 33 * 20 + 8 * 8


def _call(accumulate, n_params, fwd, bwd):
    """Runs the pair; returns its outputs."""
    f32 = dict(dtype=torch.float32, device="cuda")
    vis = torch.empty(P, dtype=torch.int64, device="cuda")
    col, logp = torch.empty(P, 3, **f32), torch.empty(P, **f32)
    fwd(vis, col, logp)
    gm = torch.full((n_params,), 0.25, **f32)
    bwd(vis, col, torch.ones(P, 3, **f32), torch.ones(P, **f32), gm)
    torch.cuda.synchronize()
    assert bool((vis == -1).all()) and bool((logp == 0).all())
    assert bool((col == torch.tensor([0.1, 0.2, 0.3], **f32)).all())
    assert bool((gm == (0.25 if accumulate else 0.0)).all())


@pytest.mark.parametrize("reuse", [0, 1])
@pytest.mark.parametrize("accumulate", [0, 1])
@pytest.mark.parametrize("dims", [[8, 16, 4], [16, 32, 32, 4], [32, 64, 64, 4]], ids=lambda d: "-".join(map(str, d)))
def test_grid_form(dims, accumulate, reuse):
    from paper_2603_27151_amd import _lib, raster as R
    ctx, h = _lib.Ctx(torch.cuda.current_device()), _lib._Holder()
    scene = _lib.soup_scene(0, 4, dims[0], len(dims) - 1, h.arr(np.asarray(dims, np.int32), C.c_int32), None, None, None)
    views = R.Views.from_list(VIEWS).c_struct(h)
    opts = _lib.make_opts(seed=3, background=(0.1, 0.2, 0.3), accumulate=accumulate, reuse_bins=reuse)
    g = torch.zeros(64, dtype=torch.float32, device="cuda")   # vertex and texture gradients: no entries
    _call(accumulate, sum(o * i + o for i, o in zip(dims[:-1], dims[1:])),
          lambda vis, col, logp: _lib.soup_rasterize_fwd(ctx, scene, views, opts, vis, col, logp),
          lambda vis, col, gc, gl, gm: _lib.soup_rasterize_bwd(ctx, scene, views, opts, vis, col, gc, gl, g, g, gm))
    ctx.close()


@pytest.mark.parametrize("accumulate", [0, 1])
@pytest.mark.parametrize("R,levels", [(0, None), (3, None), (5, None), (6, None), (5, (2, 4)), (5, (3, 5)), (6, (2, 4))])
def test_paper_form(R, levels, accumulate):
    from paper_2603_27151_amd import _lib, raster
    ctx, h = _lib.Ctx(torch.cuda.current_device()), _lib._Holder()
    scene = _lib.soup_pscene(0, R, None, None, None)
    vs = raster.Views.from_list(VIEWS)
    views, minv = vs.c_struct(h), raster.inv_view_proj(vs)
    opts = _lib.make_opts(seed=3, background=(0.1, 0.2, 0.3), accumulate=accumulate)
    fwd = lambda vis, col, logp: _lib.soup_pforward(ctx, scene, views, minv, opts, vis, col, logp)
    if levels is None:
        bwd = lambda vis, col, gc, gl, gm: _lib.soup_pbackward(ctx, scene, views, minv, opts, vis, col, gc, gl, None, None, gm)
    else:
        bwd = lambda vis, col, gc, gl, gm: _lib.soup_pbackward_levels(
            ctx, scene, views, minv, opts, vis, col, gc, gl, levels[0], None, [None] * (levels[1] - levels[0] + 1), gm)
    _call(accumulate, _lib.PMLP_PARAMS, fwd, bwd)
    ctx.close()


@pytest.mark.parametrize("R,Rmin,Rtop", [(5, 2, 4), (6, 2, 4)])
def test_no_level_arrays(R, Rmin, Rtop):
    """... and the host arrays of its levels may be NULL."""
    from paper_2603_27151_amd import _lib, raster
    ctx, h = _lib.Ctx(torch.cuda.current_device()), _lib._Holder()
    vs = raster.Views.from_list(VIEWS)
    views, minv = vs.c_struct(h), h.arr(raster.inv_view_proj(vs), C.c_float)
    opts = _lib.make_opts(background=(0.1, 0.2, 0.3))
    scene = _lib.soup_pscene(0, R, None, None, None)
    s, L, p = _lib._stream(None), _lib.lib(), _lib._ptr
    minv = C.cast(minv, C.c_void_p)

    def bwd(vis, col, gc, gl, gm):
        ctx.check(L.soup_pbackward_levels(ctx.p, C.byref(scene), C.byref(views), minv, C.byref(opts), p(vis), p(col),
                                          p(gc), p(gl), Rmin, Rtop, None, None, p(gm), s))

    _call(0, _lib.PMLP_PARAMS, lambda vis, col, logp: ctx.check(L.soup_pforward(
        ctx.p, C.byref(scene), C.byref(views), minv, C.byref(opts), p(vis), p(col), p(logp), s)), bwd)
    ctx.check(L.soup_mc_assemble(ctx.p, 0, Rmin, Rtop, R, None, None, s))
    ctx.check(L.soup_mc_assemble_bwd(ctx.p, 0, Rmin, Rtop, R, None, None, None, 0, s))
    ctx.close()

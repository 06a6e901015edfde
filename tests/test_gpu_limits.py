"""Calls of more pixels than a kernel's 32-bit indices hold are refused before any work: the pixels of a
fragment log (log p, the backwards), and the regions that the forward's waves take, with what the waves add to them. Only the refusal is exercised: nothing is launched, and the output buffers are stand-ins."""
import ctypes as C

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _views(_lib, h, sizes):
    n = len(sizes)
    return _lib.make_views(h, [w for w, _ in sizes], [hh for _, hh in sizes], np.zeros(n), np.tile(np.eye(4), (n, 1, 1)))


def _empty_scene(_lib, h):
    d = [8, 16, 4]
    return _lib.soup_scene(0, 2, 8, 2, h.arr(np.asarray(d, np.int32), C.c_int32), None, None, None)


@pytest.mark.parametrize("paper", [False, True])
def test_log_p_of_too_many_pixels(paper):
    from paper_2603_27151_amd import _lib
    ctx, h = _lib.Ctx(torch.cuda.current_device()), _lib._Holder()
    views = _views(_lib, h, [(16384, 16384)] * 16)   # 2^32 pixels
    out = torch.zeros(4, dtype=torch.int64, device="cuda")
    opts = _lib.make_opts()
    before = ctx.workspace_bytes()
    with pytest.raises(_lib.SoupError, match="2\\^32 pixels") as e:
        if paper:
            _lib.soup_pforward(ctx, _lib.soup_pscene(0, 2, None, None, None), views, np.tile(np.eye(4), (16, 1, 1)), opts,
                               out, out, out)
        else:
            _lib.soup_rasterize_fwd(ctx, _empty_scene(_lib, h), views, opts, out, out, out)
    assert e.value.status == 3 and ctx.workspace_bytes() == before
    ctx.close()


@pytest.mark.parametrize("R", [None, 5, 6])   # the grid form; the paper form sorted and per pixel
def test_backward_of_too_many_pixels(R):
    from paper_2603_27151_amd import _lib
    ctx, h = _lib.Ctx(torch.cuda.current_device()), _lib._Holder()
    views = _views(_lib, h, [(16384, 16384)] * 16)
    out = torch.zeros(4, dtype=torch.int64, device="cuda")
    before = ctx.workspace_bytes()
    with pytest.raises(_lib.SoupError, match="2\\^32 pixels") as e:
        if R is None:
            _lib.soup_rasterize_bwd(ctx, _empty_scene(_lib, h), views, _lib.make_opts(), *[out] * 7)
        else:
            _lib.soup_pbackward(ctx, _lib.soup_pscene(0, R, None, None, None), views, np.tile(np.eye(4), (16, 1, 1)),
                                _lib.make_opts(), *[out] * 7)
    assert e.value.status == 3 and ctx.workspace_bytes() == before
    ctx.close()


@pytest.mark.parametrize("last", [(16384, 16384), (16384, 16376), (16384, 16361)])
def test_too_many_regions(last):
    """8-pixel tiles: 2^32 regions and up to some thousand fewer."""
    from paper_2603_27151_amd import _lib
    ctx, h = _lib.Ctx(torch.cuda.current_device()), _lib._Holder()
    ctx.set_tile(8)
    sizes = [(16384, 16384)] * 1023 + [last]
    n = sum(((w + 7) // 8) * ((hh + 7) // 8) for w, hh in sizes)
    assert (1 << 32) - 4112 <= n <= 1 << 32
    out = torch.zeros(4, dtype=torch.int64, device="cuda")
    before = ctx.workspace_bytes()
    with pytest.raises(_lib.SoupError, match="regions") as e:
        _lib.soup_render(ctx, [_empty_scene(_lib, h)] * len(sizes), _views(_lib, h, sizes), _lib.make_opts(mode=1),
                         [out] * len(sizes))
    assert e.value.status == 3 and ctx.workspace_bytes() == before
    ctx.close()

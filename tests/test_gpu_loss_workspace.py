"""The L1 + D-SSIM loss of several views with a workspace that holds one of them: static mode after an eager pass
view by view. The views then share no launches; the results are those of the shared ones (gradients and shares
per pixel: the same arithmetic; the loss: a sum in double, one rounding to float32)."""
import numpy as np
import pytest

from paper_2603_27151_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

SIZES = [(100, 80), (33, 20), (64, 128), (1, 1), (90, 90)]


def test_static_mode_after_single_views():
    from paper_2603_27151_amd import _lib, raster as R
    rng = np.random.default_rng(2)
    views = [W.View(w, h, i, np.eye(4, dtype=np.float32)) for i, (w, h) in enumerate(SIZES)]
    P = sum(w * h for w, h in SIZES)
    c, t = (torch.from_numpy(rng.random((P, 3)).astype(np.float32)).cuda() for _ in range(2))
    want = R.loss_l1_ssim(c, t, R.Views.from_list(views), ctx=_lib.Ctx(torch.cuda.current_device()))
    ctx, at = _lib.Ctx(torch.cuda.current_device()), 0
    for v in views:
        n = v.width * v.height
        R.loss_l1_ssim(c[at:at + n], t[at:at + n], R.Views.from_list([v]), ctx=ctx)
        at += n
    ctx.set_static(True)
    got = R.loss_l1_ssim(c, t, R.Views.from_list(views), ctx=ctx)
    torch.cuda.synchronize()
    assert torch.equal(got[1], want[1]) and torch.equal(got[2], want[2])
    assert abs(float(got[0]) - float(want[0])) <= 2.0 ** -24 * len(SIZES) * float(want[0])
    big = [W.View(200, 200, 0, np.eye(4, dtype=np.float32))]   # larger than any view before: refused, as ever
    x = torch.zeros(40_000, 3, device="cuda")
    with pytest.raises(_lib.SoupError, match="static mode"):
        R.loss_l1_ssim(x, x, R.Views.from_list(big), ctx=ctx)
    ctx.close()

"""The L1 + D-SSIM loss of a call whose views take 157 batches of launches: the scalar is the shares' sum in double,
rounded to float32 once (half a unit in the last place, 2^-24 relative at most), also through the allocation-free
entry point."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("seed", [1, 2, 3, 4])
def test_one_rounding(seed):
    from paper_2603_27151_amd import _lib
    rng = np.random.default_rng(seed)
    n, h = 5000, _lib._Holder()
    w, hh = rng.integers(1, 9, n), rng.integers(1, 9, n)
    views = _lib.make_views(h, w, hh, np.zeros(n), np.tile(np.eye(4), (n, 1, 1)))
    P = int((w * hh).sum())
    c, t = (torch.from_numpy(rng.random((P, 3)).astype(np.float32)).cuda() for _ in range(2))
    ctx = _lib.Ctx(torch.cuda.current_device())
    for fn in (_lib.soup_loss_l1_ssim, _lib.soup_loss_l1_ssim_noalloc):
        gc, gl, loss = torch.empty_like(c), torch.empty(P, device="cuda"), torch.empty(1, device="cuda")
        fn(ctx, c, t, views, 0.8, gc, gl, loss)
        ref = float(gl.double().sum())
        assert abs(float(loss) - ref) <= 1.001 * 2.0 ** -24 * ref
    ctx.close()

"""The L1 + D-SSIM loss where its views spread over several batches of launches (more than 32 views, more
pixels than the records hold) and over fewer and more tiles than workgroups: every view's gradients and score
weights, scaled by the pixel counts, are those of the view alone, and the loss is the shares' sum in float64.
The oracle holds a view alone (test_gpu_train.py)."""
import numpy as np
import pytest

from paper_2603_27151_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("sizes", [[(20 + i % 7, 13 + i % 5) for i in range(70)], [(1, 1)] * 33,
                                   [(1701, 1203), (33, 9), (1703, 1201), (900, 1000)]])
def test_batches(sizes):
    from paper_2603_27151_amd import raster as R
    vs = lambda s: R.Views.from_list([W.View(w, h, 0, np.eye(4, dtype=np.float32)) for w, h in s])
    gen = torch.Generator(device="cuda").manual_seed(2)
    P = sum(w * h for w, h in sizes)
    c, t = (torch.rand(P, 3, device="cuda", generator=gen) for _ in range(2))
    loss, gc, gl = R.loss_l1_ssim(c, t, vs(sizes))
    ref = float(gl.double().sum())
    assert abs(float(loss) - ref) <= 2e-7 * abs(ref)   # one rounding to float32 and the sum's order in float64
    at = 0
    for w, h in sizes:
        s = slice(at, at + w * h)
        at = s.stop
        _, g1, l1 = R.loss_l1_ssim(c[s], t[s], vs([(w, h)]))
        k = w * h / P
        for a, b in ((gc[s], g1), (gl[s], l1)):   # the same sums, scaled by two roundings of 1 / (3 P)
            assert torch.all((a.double() - b.double() * k).abs() <= 1e-6 * b.double().abs().max() * k)

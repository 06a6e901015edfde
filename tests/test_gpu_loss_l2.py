"""The L2 loss: sizes on both sides of where its first launch begins and of its groups of four pixels, aligned
and not, with and without the scalar, against float64; and calls on two streams through one context, which must
not see each other.

Tolerances, in u = 2^-24: d has 1 rounding, 1 / (3P) has 3 (P to float32, times 3, the quotient), so 2 d / (3P)
has 5; d^2 twice d's, 3 roundings of the sum, 1 / (3P) and the product: 9; the sum of the shares is in double."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

U = 2.0 ** -24


@pytest.mark.parametrize("shift", [0, 1])   # floats from a 16-byte boundary
@pytest.mark.parametrize("P", [1, 2, 5, 1023, 4095, 4096, 4097, 4099, 5000, 300_001, 2_100_000])
def test_against_float64(P, shift):
    from paper_2603_27151_amd import raster as R
    rng = np.random.default_rng(P)
    c, t = (rng.random((P, 3)).astype(np.float32) for _ in range(2))

    def dev(n, a=None):
        x = torch.full((n + shift,), float("nan"), device="cuda")[shift:]
        return x if a is None else x.copy_(torch.from_numpy(a.reshape(-1)))

    cd, td = dev(3 * P, c).view(P, 3), dev(3 * P, t).view(P, 3)
    d = c.astype(np.float64) - t
    gc64, gl64 = 2 * d / (3 * P), (d * d).sum(1) / (3 * P)
    for with_loss in (True, False):
        loss = torch.full((1,), float("nan"), device="cuda") if with_loss else None
        gc, gl = dev(3 * P).view(P, 3), dev(P)
        R.loss_l2(cd, td, out=(loss, gc, gl))
        assert np.all(np.abs(gc.cpu().numpy() - gc64) <= 6 * U * np.abs(gc64))
        assert np.all(np.abs(gl.cpu().numpy() - gl64) <= 10 * U * gl64)
        if with_loss:
            assert abs(float(loss) - gl64.sum()) <= 11 * U * gl64.sum()


def test_two_streams_of_one_context():
    from paper_2603_27151_amd import raster as R
    P, n = 200_000, 400
    rng = np.random.default_rng(1)
    c = torch.from_numpy(rng.random((P, 3)).astype(np.float32)).cuda()
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    targets = [c + 0.25, c - 2.0]
    outs = [(torch.zeros(n, device="cuda"), torch.empty_like(c), torch.empty(P, device="cuda")) for _ in streams]
    alone = []
    for t, (loss, gc, gl) in zip(targets, outs):
        R.loss_l2(c, t, out=(loss[:1], gc, gl))
        alone.append(float(loss[0]))
    torch.cuda.synchronize()
    x = torch.ones(8192, 8192, device="cuda")
    for _ in range(20):   # both streams wait for this, so that their calls are queued and then run side by side
        x = x @ x * 1e-4
    for s in streams:
        s.wait_stream(torch.cuda.current_stream())
    for i in range(n):
        for s, t, (loss, gc, gl) in zip(streams, targets, outs):
            R.loss_l2(c, t, stream=s, out=(loss[i:i + 1], gc, gl))
    torch.cuda.synchronize()
    for a, (loss, _, _) in zip(alone, outs):
        assert bool((loss == a).all()), f"{int((loss != a).sum())} of {n} losses differ"

"""The decoder's float32 sequence on the matrix cores, where any other order shows.

First-layer weights come in pairs (w, -w) over channels that are equal up to a few ulps, so every
first-layer pre-activation is what rounding leaves of a sum that cancels: its sign, and with it the
ReLU decision, depends on the order and the rounding of every step. The visibility (drawn against
the decoded opacity) is held bit for bit, the gradients (through the recomputed ReLU decisions) to
the bounds of tests/parity.py. Sizes leave a single fragment, a few, and ragged batches of 64.
"""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2603_27151_amd import workloads as W
from tests import parity as PT

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _scene(dims, G, T, seed):
    rng = np.random.Generator(np.random.PCG64(seed))
    s = W.random_scene(rng, W.equilateral_soup(rng, W.uniform_ball(rng, T, 0.3), log_mean=-1.0), G, dims[0], dims)
    f = s.feats.reshape(-1, dims[0])
    f *= 20.0
    f[:, 1::2] = f[:, 0::2] * (1 + rng.integers(-2, 3, f[:, 0::2].shape).astype(np.float32) * np.float32(2.0 ** -23))
    w0 = s.mlp[:dims[0] * dims[1]].reshape(dims[1], dims[0])
    w0[:, 1::2] = -w0[:, 0::2]
    at = dims[0] * dims[1] + dims[1]
    s.mlp[at:at + dims[1] * dims[2]] *= 2.0 ** 20   # brings the rounding-sized activations back to order one
    return s


@pytest.mark.parametrize("reuse", [0, 1])
@pytest.mark.parametrize("size", [(1, 1), (5, 3), (37, 29), (129, 64)])
@pytest.mark.parametrize("dims,G", [([8, 16, 4], 4), ([16, 32, 32, 4], 8), ([32, 64, 64, 4], 4)])
def test_cancelling_first_layer(dims, G, size, reuse):
    from paper_2603_27151_amd import raster as R
    s = _scene(dims, G, 40, 7 + dims[0])
    v = W.View(size[0], size[1], 3, W.view_proj((0.0, 0.0, 3.0), size[0], size[1]))
    vs, oo = R.Views.from_list([v]), O.Opts(seed=11)
    ds = R.DeviceScene.from_host(s)
    opts = R.Opts(seed=11, reuse_bins=reuse)
    vis, col, _ = R.rasterize_fwd(ds, vs, opts)
    rvis, rcol, _, _ = O.forward(s, v, oo)
    assert np.array_equal(vis.cpu().numpy().view(np.uint64).reshape(rvis.shape), rvis)
    PT.assert_colours(col.cpu().numpy().reshape(rcol.shape), rcol)
    P = size[0] * size[1]
    d = rcol - np.random.default_rng(5).random(rcol.shape).astype(np.float32)
    gc = (2 * d / np.float32(3 * P)).astype(np.float32)
    gl = ((d * d).sum(-1) / np.float32(3 * P)).astype(np.float32)
    up = lambda a, k: torch.from_numpy(np.ascontiguousarray(a.reshape(-1, k) if k > 1 else a.reshape(-1))).cuda()
    got = R.rasterize_bwd(ds, vs, opts, vis, col, up(gc, 3), up(gl, 1))
    ref = O.backward(s, v, oo, rvis, rcol, gc, gl)
    # (not the vertices': their colour path sums d x_k . slope_k over the channels, and here paired channels
    # have opposite gradients and equal slopes, so that sum is rounding alone in any implementation)
    PT.assert_grads([g.cpu().numpy() for g in got[1:]], ref[1:], names=("feats", "mlp"))

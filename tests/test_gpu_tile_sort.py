"""The tile lists' sort where its variants meet: one wave up to 256 entries, a workgroup with 512, 1,024 and
2,048 in registers, lists of several blocks with every kind of last block. Every pixel of a small view has
the same list of T entries and walks deep into it (a low opacity); its early exit trusts the order."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2603_27151_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("T", [2, 33, 300, 511, 512, 513, 1023, 1024, 1025, 2047, 2048, 2049, 2112, 2113, 2304, 2305, 4097])
def test_sizes(T):
    from paper_2603_27151_amd import raster as R
    rng = np.random.default_rng(7000 + T)
    ang = rng.uniform(0.0, 2.0 * np.pi, T)[:, None] + np.array([0.0, 2.0 * np.pi / 3.0, 4.0 * np.pi / 3.0])
    verts = np.stack([4.0 * np.cos(ang), 4.0 * np.sin(ang), rng.uniform(-0.2, 0.2, (T, 3))], axis=2)
    verts = (verts + W.uniform_ball(rng, T, 0.5)[:, None, :]).astype(np.float32)
    verts[1::7] = verts[::7][:len(verts[1::7])]          # equal depth bounds
    s = W.random_scene(rng, verts, 4, 8, [8, 16, 4])
    s.mlp[-1] = -5.0
    v = W.View(16, 8, 1, W.view_proj((0.0, 0.0, 3.0), 16, 8))
    vis, _, _ = R.rasterize_fwd(R.DeviceScene.from_host(s), R.Views.from_list([v]), R.Opts(seed=3))
    assert np.array_equal(vis.cpu().numpy().view(np.uint64).reshape(8, 16), O.forward(s, v, O.Opts(seed=3))[0])

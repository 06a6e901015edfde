"""The forward's coverage masks, in 32-bit integers, where they can go wrong: edges exactly through
pixel centres (both windings, shared edges), vertices on the snapping grid, edges of triangles far
larger than the image up to the largest coordinates, slivers, and pixels whose best key has the same
depth. The visibility has to be the oracle's, whole value by whole value."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2603_27151_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

SIZE = 64   # a power of two: pixel coordinates map onto clip coordinates exactly


def _triangles(kind, rng, T):
    if kind == "centres":
        p = rng.integers(-8, SIZE + 8, (T, 3, 2)) + 0.5
    elif kind == "shared":   # quads with corners at centres, cut along both diagonals, both windings
        a = rng.integers(0, SIZE - 9, (T // 2, 2)) + 0.5
        d = rng.integers(1, 9, (T // 2, 2))
        q = np.stack([a, a + d * [1, 0], a + d, a + d * [0, 1]], 1)
        p = np.concatenate([q[:, [0, 1, 2]], q[:, [2, 0, 3]]])
        p[::3] = p[::3, ::-1]
    elif kind == "grid":
        p = rng.integers(-256 * 8, 256 * (SIZE + 8), (T, 3, 2)) / 256.0
    elif kind == "far":
        p = rng.integers(-65535, 65536, (T, 3, 2)) + rng.integers(0, 256, (T, 3, 2)) / 256.0
        p = np.clip(p, -65535.0, 65535.0)
        p[::4, 0] = [-65535.0, -65535.0]
        p[::4, 1] = [65535.0, 65535.0]
        p[1::4, 0] = [0.5, -65535.0]
    else:   # slivers
        a = rng.integers(0, 256 * SIZE, (T, 2)) / 256.0
        p = np.stack([a, a + rng.integers(-4000, 4001, (T, 2)) / 256.0, a + rng.integers(-3, 4, (T, 2)) / 256.0], 1)
    return p


@pytest.mark.parametrize("kind", ["centres", "shared", "grid", "far", "slivers"])
@pytest.mark.parametrize("flat", [False, True])
def test_masks(kind, flat):
    from paper_2603_27151_amd import raster as R
    rng = np.random.Generator(np.random.PCG64(17))
    T = 200
    p = _triangles(kind, rng, T)
    z = np.zeros((p.shape[0], 3)) if flat else rng.uniform(-0.9, 0.9, (p.shape[0], 3))
    verts = np.concatenate([p / (SIZE / 2) * [1.0, -1.0] + [-1.0, 1.0], z[..., None]], 2)
    s = W.random_scene(rng, verts, 4, 8, [8, 16, 4])
    v = W.View(SIZE, SIZE, 3, np.eye(4, dtype=np.float32))
    o = O.Opts(seed=11)
    rvis, _, _, _ = O.forward(s, v, o)
    vis, _, _ = R.rasterize_fwd(R.DeviceScene.from_host(s), R.Views.from_list([v]), R.Opts(seed=11))
    got = vis.cpu().numpy().view(np.uint64).reshape(rvis.shape)
    assert (rvis != np.uint64(0xFFFFFFFFFFFFFFFF)).any()
    assert np.array_equal(got, rvis)


@pytest.mark.parametrize("size", [(13, 9), (1, 1), (31, 17)])
def test_covered_pixels_at_the_near_plane(size):
    """Triangles of depth 0 over views that end inside a block: the pixels counted as covered are the view's."""
    from paper_2603_27151_amd import _lib, raster as R
    rng = np.random.Generator(np.random.PCG64(4))
    verts = np.array([[[-3.0, -1.0, -1.0], [3.0, -1.0, -1.0], [0.0, 5.0, -1.0]]] * 3)
    s = W.random_scene(rng, verts, 4, 8, [8, 16, 4])
    v = W.View(size[0], size[1], 3, np.eye(4, dtype=np.float32))
    ctx = _lib.Ctx(torch.cuda.current_device())
    ctx.set_counting(True)
    vis, _, _ = R.rasterize_fwd(R.DeviceScene.from_host(s), R.Views.from_list([v]), R.Opts(seed=2), ctx=ctx)
    assert np.array_equal(vis.cpu().numpy().view(np.uint64).reshape(size[1], size[0]), O.forward(s, v, O.Opts(seed=2))[0])
    assert ctx.stats()["covered_pixels"] == size[0] * size[1]

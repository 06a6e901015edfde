"""The backward decode of short fragment lists, whose waves take ranges in blocks of 16 fragments: from
no fragment and one to a few per wave, ranges that end inside a batch and inside a block, triangles
of all of a list and of a few fragments, all decoder shapes. Oracle and tolerances are those of the
forward and backward's parity."""
import numpy as np
import pytest

from paper_2603_27151_amd import workloads as W

from . import test_gpu_parity as parity

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims", [[8, 16, 4], [16, 32, 32, 4], [32, 64, 64, 4]], ids=lambda d: "-".join(map(str, d)))
@pytest.mark.parametrize("T,sizes", [(1, [(1, 1)]), (3, [(4, 4)]), (2, [(5, 3), (17, 1)]), (40, [(9, 8)]), (5, [(64, 50)]),
                                     (400, [(97, 61), (31, 33)])])
def test_short_lists(dims, T, sizes):
    rng = np.random.Generator(np.random.PCG64(T))
    verts = W.equilateral_soup(rng, W.uniform_ball(rng, T, 0.5), log_mean=0.5 if T <= 5 else -1.0)
    scene = W.random_scene(rng, verts, 4, dims[0], dims)
    views = [W.View(w, h, i, W.view_proj((0.0, 0.0, 3.0), w, h)) for i, (w, h) in enumerate(sizes)]
    parity._fwd_bwd_case(W.Workload("short", scene, views, 77))

"""The bottom-up step of the GPU linear-BVH builder and the four-child merge.

The step completes the subtrees within runs of 512 sorted leaves, then of
16,384, then of 524,288, and then the rest; the merge expands subtrees in a
workgroup's list and hands nodes on when the list outgrows its threads.  The
sizes lie on both sides of each run, the scenes give balanced, skewed and
depth-limited trees.  The structure is checked exactly and hits against brute
force bit for bit.
"""
import sys

import numpy as np
import pytest

from bvh_structure import check_structure
from paper_1505_06022_amd import api, scenes

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    return torch


def _skewed(n):
    """Centres at powers of two: most of the triangles share few cells, the tree is deep and uneven."""
    rng = np.random.default_rng(n)
    v = (2.0 ** -(np.arange(n) % 22)).astype(np.float32)[:, None, None] * rng.uniform(0.9, 1.0, (n, 3, 3))
    return v.astype(np.float32)


def _soup(n):
    return scenes.small_soup(n, n % 13, spread=0.4 / max(1.0, np.cbrt(n))).verts


@pytest.mark.parametrize("make,n,max_leaf", [(_soup, 511, 4), (_soup, 512, 1), (_soup, 513, 4), (_soup, 1025, 7),
                                             (_soup, 16384, 4), (_soup, 16385, 4), (_soup, 16897, 1),
                                             (_skewed, 3000, 1), (_skewed, 20000, 4)])
def test_runs(torch_cuda, oracle_lib, make, n, max_leaf):
    print(f"case: GPU LBVH runs {make.__name__} n={n} max_leaf={max_leaf}", flush=True)
    sys.stdout.flush()
    verts = make(n)
    mats = (np.arange(n) % 5).astype(np.uint32)
    bvh = api.build_bvh(verts, mats, max_leaf=max_leaf, builder=api.BUILD_GPU_LBVH)
    info = bvh.info()
    nodes, tris = bvh.download()
    assert check_structure(verts, nodes, tris, max_leaf, info)
    assert np.array_equal(tris[:, 10], mats[tris[:, 9]])
    rays = scenes.random_rays(1500, n)
    h_ref, t_ref = oracle_lib.trace_brute_force(verts, rays)
    h, t = api.trace_rays(bvh, torch_cuda.from_numpy(rays).cuda())
    h, t = h.cpu().numpy(), t.cpu().numpy()
    assert np.array_equal(h, h_ref)
    assert np.array_equal(t[h_ref >= 0], t_ref[h_ref >= 0])
    bvh.destroy()


def test_past_the_third_run(torch_cuda):
    """524,289 triangles: the hits of the SAH BVH."""
    n = 524_289
    print(f"case: GPU LBVH n={n}", flush=True)
    verts = _soup(n)
    rays = torch_cuda.from_numpy(scenes.random_rays(100_001, 4)).cuda()
    out = []
    for builder in (api.BUILD_HOST_SAH, api.BUILD_GPU_LBVH):
        bvh = api.build_bvh(verts, None, builder=builder)
        out.append([x.cpu().numpy() for x in api.trace_rays(bvh, rays)])
        bvh.destroy()
    assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])


@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan])
def test_non_finite_vertex_is_named(torch_cuda, bad):
    print(f"case: GPU LBVH vertex {bad}", flush=True)
    verts = _soup(700)
    verts[613, 2, 1] = bad
    with pytest.raises(Exception, match="triangle 613"):
        api.build_bvh(verts, None, builder=api.BUILD_GPU_LBVH)

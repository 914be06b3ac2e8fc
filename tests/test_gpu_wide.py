"""The four-child walk against the oracle's brute force: wave and quad
remainders, ragged tiles, trees that run its stack out or are too deep for it.
The walk tests the same boxes and triangles as the binary one, so hit index and
t are equal bit for bit (tolerance 0)."""
import numpy as np
import pytest

from paper_1505_06022_amd import api, scenes

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    return torch


def _chain(n, ratio, top):
    """n triangles facing -x, at x = top ratio^-i and as large as that: each
    group of the smaller ones lies in front of the next, so the tree (two bins)
    is a chain and a ray along +x finds the inner child nearest at every level."""
    k = top * float(ratio) ** np.arange(1 - n, 1.0)
    tri = np.array([[0, -1, -1], [0, 2, -1], [0, -1, 2]], np.float64)
    v = k[:, None, None] * tri[None]
    v[:, :, 0] += k[:, None]
    return v.astype(np.float32)


def _wide_depth(verts, **opts):
    """Levels of four-child nodes: the host build's binary tree, opened largest box first."""
    nodes, _, info = api.build_bvh_host(verts, None, **opts)
    q = nodes[0]
    step = np.asarray(info["grid_step"], np.float64)
    ext = ((q[:, :3] >> 16).astype(np.int64) - (q[:, :3] & 0xffff)) * step
    area = ext[:, 0] * ext[:, 1] + ext[:, 1] * ext[:, 2] + ext[:, 2] * ext[:, 0]
    leaf = (q[:, 3] >> 31) != 0
    level, depth = [0], 0
    while level:
        nxt = []
        for v in level:
            kids = [v]
            while len(kids) < 4:
                inner = [k for k in kids if not leaf[k]]
                if not inner:
                    break
                o = max(inner, key=lambda k: area[k])
                kids[kids.index(o)] = o + 1
                kids.append(o + 2 if leaf[o + 1] else int(q[o + 1, 3]))
            nxt += [k for k in kids if not leaf[k]]
        level, depth = nxt, depth + 1
    return depth


def _check(torch_cuda, oracle_lib, verts, rays, calls, **opts):
    bvh = api.build_bvh(verts, np.zeros(len(verts), np.uint32), **opts)
    h_ref, t_ref = oracle_lib.trace_brute_force(verts, rays)
    r = torch_cuda.from_numpy(rays).cuda()
    for kw in calls:
        print("case:", len(verts), len(rays), kw, flush=True)
        h, t = api.trace_rays(bvh, r, **kw)
        assert np.array_equal(h.cpu().numpy(), h_ref), kw
        assert np.array_equal(t.cpu().numpy(), t_ref), kw
    return h_ref


@pytest.mark.parametrize("n", [1, 15, 16, 17, 63, 64, 65, 1009, 65535, 65536, 65537])
def test_ray_counts(torch_cuda, oracle_lib, n):
    sc = scenes.small_soup(200, 4)
    rays = scenes.random_rays(n, 5)
    rays[::7, 3] = -2.0            # hits behind the origin count down to tmin
    rays[::11, 7] = 0.3
    rays[::13, 4:7] = (0, 0, 1)    # axis-parallel
    calls = [dict(), dict(block=128), dict(kernel=api.TRACE_POSTPONED, refill=32, reorder=1, block=64),
             dict(kernel=api.TRACE_POSTPONED, refill=0), dict(kernel=api.TRACE_PACKET, reorder=2)]
    _check(torch_cuda, oracle_lib, sc.verts, rays, calls)


@pytest.mark.parametrize("size", [(1, 1), (7, 9), (8, 8), (13, 21), (333, 199)])
def test_ragged_tiles(torch_cuda, oracle_lib, size):
    w, h = size
    sc = scenes.box_scene(w, h)
    rays = scenes.pinhole_rays(sc.camera)
    _check(torch_cuda, oracle_lib, sc.verts, rays,
           [dict(kernel=api.TRACE_PACKET, tile_width=w, block=64), dict(tile_width=w)])


@pytest.mark.parametrize("tris", [1, 2, 3, 4, 5, 17])
def test_smallest_trees(torch_cuda, oracle_lib, tris):
    sc = scenes.small_soup(tris, 6)
    for leaf in (1, 4, 7):
        for builder in (api.BUILD_HOST_SAH, api.BUILD_GPU_LBVH):
            _check(torch_cuda, oracle_lib, sc.verts, scenes.random_rays(500, 7), [dict()], max_leaf=leaf,
                   builder=builder)


@pytest.mark.parametrize("n,ratio,top,levels", [(300, 1.15, 1e9, (20, 32)), (500, 1.15, 1e12, (33, 99))])
def test_deep_trees(torch_cuda, oracle_lib, n, ratio, top, levels):
    """Chains whose rays push leaves at every level, more than the stack holds (20 to 32 levels), and one with more
    levels than the four-child nodes are built for (32)."""
    opts = dict(max_leaf=1, bins=2)
    verts = _chain(n, ratio, top)
    assert levels[0] <= _wide_depth(verts, **opts) <= levels[1]
    rng = np.random.default_rng(3)
    m = 400
    rays = np.zeros((m, 8), np.float32)
    rays[:, 1:3] = rng.uniform(-0.3, 0.3, (m, 2)) * float(verts[0].max())
    rays[:, 4] = 1.0
    rays[:, 5:7] = rng.uniform(-0.2, 0.2, (m, 2))
    rays[:, 7] = np.inf
    rays[:, 3] = top * float(ratio) ** rng.integers(-n, 0, m)  # past the first triangles
    h = _check(torch_cuda, oracle_lib, verts, rays,
               [dict(), dict(kernel=api.TRACE_POSTPONED, refill=16, reorder=1), dict(kernel=api.TRACE_PER_RAY)], **opts)
    assert len(np.unique(h)) > n // 4


@pytest.mark.parametrize("scale", [1e-9, 1e-3, 1e3, 1e7, 1e9])
def test_scene_scales(torch_cuda, oracle_lib, scale):
    """Axis-parallel rays (zero direction components) in scenes of any size, with every kernel."""
    sc = scenes.box_scene()
    verts = (sc.verts * np.float32(scale)).astype(np.float32)
    rays = scenes.random_rays(3000, 9)
    rays[:, :3] = (rays[:, :3] * np.float32(0.98) + np.float32(0.01)) * np.float32(scale)
    for a in range(3):
        rays[a::6, 4:7] = np.eye(3, dtype=np.float32)[a]
        rays[a + 3::6, 4 + a] = 0.0
    rays[5::9, 4:7] *= -1.0
    rays[::17, 4] = np.float32(1e-33)  # a tiny component beside a larger one
    rays[::17, 5] = 0.7
    _check(torch_cuda, oracle_lib, verts, rays,
           [dict(), dict(kernel=api.TRACE_POSTPONED, refill=8, reorder=1)] + [dict(kernel=k) for k in (1, 2, 3, 5, 6)])

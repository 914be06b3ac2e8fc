"""Four-child nodes merged on the host (small trees) and on the device, both
builders, at the sizes where the way changes, and trees too deep for them: the
default walk gives the binary walk's hits bit for bit."""
import numpy as np
import pytest

from paper_1505_06022_amd import api, scenes
from test_gpu_wide import _chain, _wide_depth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    return torch


def _compare(torch_cuda, bvh, rays):
    r = torch_cuda.from_numpy(rays).cuda()
    ref = api.trace_rays(bvh, r, kernel=api.TRACE_PER_RAY)
    for kw in (dict(), dict(kernel=api.TRACE_POSTPONED, refill=16, reorder=1)):
        got = api.trace_rays(bvh, r, **kw)
        assert torch_cuda.equal(ref[0], got[0]) and torch_cuda.equal(ref[1], got[1]), kw
    return ref[0]


@pytest.mark.parametrize("builder", [api.BUILD_HOST_SAH, api.BUILD_GPU_LBVH])
@pytest.mark.parametrize("tris", [1, 2, 5, 36, 900, 1_000, 8_200, 8_300, 8_400, 8_600, 9_000])
def test_sizes(torch_cuda, tris, builder):
    print("case: small tree", tris, "builder", builder, flush=True)
    sc = scenes.small_soup(tris, 2, spread=0.05)
    bvh = api.build_bvh(sc.verts, sc.tri_mat, builder=builder)
    hit = _compare(torch_cuda, bvh, scenes.random_rays(70_000, 3))
    assert tris < 36 or int(hit.max()) >= 0


@pytest.mark.parametrize("n,ratio", [(500, 1.15), (4200, 1.02)])
def test_too_deep(torch_cuda, n, ratio):
    opts = dict(max_leaf=1, bins=2)
    verts = _chain(n, ratio, 1e12)
    assert _wide_depth(verts, **opts) > 32
    print("case: deep tree", n, flush=True)
    rng = np.random.default_rng(3)
    rays = np.zeros((70_000, 8), np.float32)
    rays[:, 4], rays[:, 7] = 1.0, np.inf
    rays[:, 5:7] = rng.uniform(-0.2, 0.2, (70_000, 2))
    rays[:, 3] = 1e12 * ratio ** rng.integers(-n, 0, 70_000).astype(np.float64)
    hit = _compare(torch_cuda, api.build_bvh(verts, np.zeros(n, np.uint32), **opts), rays)
    assert len(np.unique(hit.cpu().numpy())) > 100

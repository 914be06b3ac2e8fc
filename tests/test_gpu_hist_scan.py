"""The bucket starts of the bucketed trace: rays in few buckets, in many, and in the last, give the hits of the input order."""
import numpy as np
import pytest

from paper_1505_06022_amd import api, scenes

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    return torch


@pytest.mark.parametrize("n", [1, 65, 4097, 100_003])
@pytest.mark.parametrize("spread", ["all", "one", "corner"])
def test_bucketed_equals_input_order(torch_cuda, n, spread):
    torch = torch_cuda
    print("case: bucket scan", n, spread, flush=True)
    sc = scenes.small_soup(3000, 5, spread=0.03)
    bvh = api.build_bvh(sc.verts, sc.tri_mat)
    rays = scenes.random_rays(n, 3)
    if spread == "one":
        rays[:, :3] = rays[0, :3]
        rays[:, 4:7] = rays[0, 4:7]
    elif spread == "corner":  # beyond the scene's last cell along every axis, towards -z: the last bucket
        rays[:, :3] = 10.0
        rays[:, 4:7] = -10.0 + rays[:, 4:7]
        rays[:, 6] -= 5.0
    r = torch.from_numpy(np.ascontiguousarray(rays)).cuda()
    h0, t0 = api.trace_rays(bvh, r)
    for kw in (dict(kernel=api.TRACE_POSTPONED, refill=32, reorder=1, block=64), dict(kernel=api.TRACE_PER_RAY, reorder=1)):
        h, t = api.trace_rays(bvh, r, torch.full_like(h0, -7), torch.full_like(t0, -7.0), **kw)
        assert torch.equal(h, h0) and torch.equal(t, t0), kw

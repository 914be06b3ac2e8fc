"""Iterations that overlap on the device give what iterations waited for one by one give, bit for bit."""
import numpy as np
import pytest

from paper_1505_06022_amd import api, scenes

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    return torch


@pytest.mark.parametrize("gather", [api.GATHER_EXACT, api.GATHER_STOCHASTIC])
def test_one_call_equals_single_iterations(torch_cuda, gather):
    """The stochastic gather reads the photon store itself, the exact one a sorted copy: neither may see the photons
    of a later pass in that store."""
    sc = scenes.procedural_scene(width=640, height=360, hf_cells=60, sphere_level=3, glass_level=4, seed=11)
    print("case: overlap, gather", gather, flush=True)
    p = api.sppm_params(20_001, r0=0.02, seed=3, gather_mode=gather)
    bvh = api.build_bvh(sc.verts, sc.tri_mat)
    one, many = api.Sppm(sc, p, bvh=bvh), api.Sppm(sc, p, bvh=bvh)
    one.iterate(12)
    for _ in range(12):
        many.iterate(1)
        torch_cuda.cuda.synchronize()
    a, b = one.views(), many.views()
    torch_cuda.cuda.synchronize()
    for key in ("N", "R2", "tau", "D"):
        assert np.array_equal(a[key].cpu().numpy(), b[key].cpu().numpy()), key
    assert torch_cuda.equal(one.resolve(), many.resolve())

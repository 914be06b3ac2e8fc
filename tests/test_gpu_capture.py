"""A call of several iterations, and of the adjoint, recorded into a graph: the streams that the call uses join the caller's."""
import pytest

from paper_1505_06022_amd import api, scenes

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    return torch


@pytest.mark.parametrize("photons", [20_001, 270_001])
@pytest.mark.parametrize("n", [1, 2, 5])
def test_iterations_and_adjoint_under_capture(torch_cuda, photons, n):
    torch = torch_cuda
    print("case: capture, photons", photons, "iterations", n, flush=True)
    sc = scenes.procedural_scene(width=96, height=61, hf_cells=40, sphere_level=2, glass_level=3, seed=5)
    bvh = api.build_bvh(sc.verts, sc.tri_mat)
    p = api.sppm_params(photons, r0=0.03, seed=3, record_iterations=n)
    eager, taped = api.Sppm(sc, p, bvh=bvh), api.Sppm(sc, p, bvh=bvh)
    mats = [m for m in range(len(sc.mat_rho)) if sc.mat_rho[m] > 0.0]
    g = torch.linspace(-1.0, 2.0, 96 * 61, device="cuda")
    eager.iterate(n)
    ref, ref_grad = eager.resolve(), eager.adjoint(g, mats)
    image = torch.empty_like(ref)
    grad = torch.empty_like(ref_grad)
    torch.cuda.synchronize()
    forward, backward = torch.cuda.CUDAGraph(), torch.cuda.CUDAGraph()
    with torch.cuda.graph(forward):
        taped.iterate(n, stream=torch.cuda.current_stream())
        taped.resolve(image, stream=torch.cuda.current_stream())
    with torch.cuda.graph(backward):
        taped.adjoint(g, mats, grad, stream=torch.cuda.current_stream())
    forward.replay()
    torch.cuda.synchronize()
    assert torch.equal(image, ref)
    for _ in range(3):  # the adjoint changes nothing that it reads
        grad.zero_()
        backward.replay()
        torch.cuda.synchronize()
        assert torch.equal(grad, ref_grad)

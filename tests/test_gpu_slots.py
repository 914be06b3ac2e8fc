"""The last photons and hit points of overlapped iterations against a handle that
runs one at a time, record by record, and calls of every photon schedule recorded
into a graph."""
import numpy as np
import pytest

from paper_1505_06022_amd import api, scenes

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    return torch


def _last(s):
    v = s.views()
    n = int(v["photon_count"][0])
    ph = v["photons"][:n].cpu().numpy()
    return ph[np.argsort(ph[:, 7].view(np.uint32), kind="stable")], v["hp_pos"].cpu().numpy(), v["hp_nrm"].cpu().numpy()


@pytest.mark.parametrize("photons", [20_001, 270_001])
@pytest.mark.parametrize("gather", [api.GATHER_EXACT, api.GATHER_STOCHASTIC])
def test_photons_and_hit_points(torch_cuda, photons, gather):
    print("case: slots, photons", photons, "gather", gather, flush=True)
    sc = scenes.procedural_scene(width=160, height=91, hf_cells=60, sphere_level=3, glass_level=4, seed=11)
    bvh = api.build_bvh(sc.verts, sc.tri_mat)
    serial = api.Sppm(sc, api.sppm_params(photons, r0=0.03, seed=3, gather_mode=gather, profile=api.PROFILE_TIME), bvh=bvh)
    ring = api.Sppm(sc, api.sppm_params(photons, r0=0.03, seed=3, gather_mode=gather), bvh=bvh)
    for n in (1, 2, 3, 5):
        for s in (serial, ring):
            s.iterate(n)
            s.status()
        for a, b in zip(_last(serial), _last(ring)):
            assert np.array_equal(a.view(np.uint32), b.view(np.uint32)), n


@pytest.mark.parametrize("kw", [dict(photon_kernel=k) for k in range(1, 7)] +
                         [dict(single_link_set=2), dict(photon_kernel=6, single_link_set=2),
                          dict(gather_mode=api.GATHER_STOCHASTIC)], ids=str)
def test_under_capture(torch_cuda, kw):
    torch = torch_cuda
    print("case: capture", kw, flush=True)
    sc = scenes.procedural_scene(width=96, height=61, hf_cells=40, sphere_level=2, glass_level=3, seed=5)
    bvh = api.build_bvh(sc.verts, sc.tri_mat)
    n = 4
    rec = 0 if "gather_mode" in kw else n
    p = api.sppm_params(20_001, r0=0.03, seed=3, record_iterations=rec, **kw)
    eager, taped = api.Sppm(sc, p, bvh=bvh), api.Sppm(sc, p, bvh=bvh)
    mats = [m for m in range(len(sc.mat_rho)) if sc.mat_rho[m] > 0.0]
    g = torch.linspace(-1.0, 2.0, 96 * 61, device="cuda")
    eager.iterate(n)
    ref = eager.resolve()
    image = torch.empty_like(ref)
    forward, backward = torch.cuda.CUDAGraph(), torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(forward):
        taped.iterate(n, stream=torch.cuda.current_stream())
        taped.resolve(image, stream=torch.cuda.current_stream())
    forward.replay()
    torch.cuda.synchronize()
    assert torch.equal(image, ref)
    if rec:
        want = eager.adjoint(g, mats)
        grad = torch.empty_like(want)
        with torch.cuda.graph(backward):
            taped.adjoint(g, mats, grad, stream=torch.cuda.current_stream())
        for _ in range(3):
            grad.zero_()
            backward.replay()
            torch.cuda.synchronize()
            assert torch.equal(grad, want)

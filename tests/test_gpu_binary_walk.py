"""The passes' binary-walk forms (one link set for every ray) against the
four-child walk: the same images, state and gradients, bit for bit, for each
photon schedule that has both, with few paths and with enough for two launches."""
import pytest

from paper_1505_06022_amd import api, scenes

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    return torch


@pytest.mark.parametrize("kernel,photons", [(0, 20_001), (0, 270_001), (1, 20_001), (2, 20_001), (3, 20_001),
                                            (6, 20_001)])
@pytest.mark.parametrize("link_set", [1, 6])
def test_equals_the_wide_walk(torch_cuda, kernel, photons, link_set):
    print("case: binary walk, photon kernel", kernel, "photons", photons, "set", link_set - 1, flush=True)
    sc = scenes.procedural_scene(width=96, height=61, hf_cells=40, sphere_level=2, glass_level=3, seed=5)
    bvh = api.build_bvh(sc.verts, sc.tri_mat)
    mats = [m for m in range(len(sc.mat_rho)) if sc.mat_rho[m] > 0.0]
    g = torch_cuda.linspace(-1.0, 2.0, 96 * 61, device="cuda")
    out = []
    for single in (0, link_set):
        s = api.Sppm(sc, api.sppm_params(photons, r0=0.03, seed=3, photon_kernel=kernel, record_iterations=4,
                                         single_link_set=single), bvh=bvh)
        s.iterate(4)
        s.status()
        v = s.views()
        out.append([v[k].clone() for k in ("N", "R2", "tau", "D")] + [s.resolve(), s.adjoint(g, mats)])
        s.destroy()
    assert float(out[0][-1].abs().max()) > 0.0
    for a, b in zip(*out):
        assert torch_cuda.equal(a, b)


@pytest.mark.parametrize("chunk", [64, 1024])
def test_batch(torch_cuda, chunk):
    """Without, with some and with all scenes on the binary walk."""
    scs = [scenes.box_scene(64, 48), scenes.procedural_scene(width=80, height=50, hf_cells=20, sphere_level=2,
                                                             glass_level=2, seed=4)]
    images = []
    for sets in ((0, 0), (0, 2), (5, 2)):
        print("case: batch, chunk", chunk, "sets", sets, flush=True)
        prm = [api.sppm_params(9_001, r0=0.05, seed=7 + i, single_link_set=k) for i, k in enumerate(sets)]
        images.append(api.render_batch(scs, prm, 3, chunk=chunk))
    for other in images[1:]:
        for a, b in zip(images[0], other):
            assert torch_cuda.equal(a, b)

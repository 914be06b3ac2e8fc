"""The default photon pass at the path counts where its split over the device
changes (16 to 64 paths a wave in one launch, then two launches), against one
path per lane: the same photons, counts and image, bit for bit."""
import numpy as np
import pytest

from paper_1505_06022_amd import api, scenes

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    return torch


def _photons(s):
    v = s.views()
    n = int(v["photon_count"][0])
    ph = v["photons"][:n].cpu().numpy()
    return n, int(v["photon_count"][2]), ph[np.argsort(ph[:, 7].view(np.uint32), kind="stable")]


@pytest.mark.parametrize("n", [1, 15, 16, 17, 63, 65_535, 65_537, 262_143, 262_144, 262_145, 300_001])
def test_default_pass_equals_one_path_per_lane(torch_cuda, n):
    sc = scenes.procedural_scene(width=24, height=20, hf_cells=10, sphere_level=1, glass_level=2, seed=2)
    print("case: paths", n, flush=True)
    bvh = api.build_bvh(sc.verts, sc.tri_mat)
    a = api.Sppm(sc, api.sppm_params(n, r0=0.03, seed=9), bvh=bvh)
    b = api.Sppm(sc, api.sppm_params(n, r0=0.03, seed=9, photon_kernel=api.PHOTON_PER_PATH), bvh=bvh)
    for s in (a, b):
        s.iterate(3)
        s.status()
    (na, handed, pa), (nb, _, pb) = _photons(a), _photons(b)
    assert na == nb and handed >= n
    assert np.array_equal(pa, pb)
    assert torch_cuda.equal(a.resolve(), b.resolve())

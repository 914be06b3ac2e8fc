"""The range query at the sizes where its split changes (4, 16 or 64 hit points
a wave) and at radii where a hit point is scanned by its lane or by the wave:
counts and fixed-point fluxes equal the oracle's (integers, tolerance 0)."""
import numpy as np
import pytest

from paper_1505_06022_amd import api, scenes

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    return torch


@pytest.mark.parametrize("size", [(1, 1), (3, 1), (5, 1), (17, 3), (128, 128), (127, 131), (512, 256), (257, 511)])
@pytest.mark.parametrize("r0", [0.004, 0.05, 0.4])
def test_hits_per_wave(torch_cuda, oracle_lib, size, r0):
    sc = scenes.box_scene(*size)
    n, seed = 3001, 7
    print("case:", size, r0, flush=True)
    s = api.Sppm(sc, api.sppm_params(n, r0=r0, seed=seed))
    s.iterate(1)
    osc = oracle_lib.OracleScene(sc)
    M, Phi = oracle_lib.gather(oracle_lib.eye_pass(osc, seed, 0), oracle_lib.photon_pass(osc, seed, 0, n),
                               np.full(osc.P, r0 * r0))
    v = s.views()
    torch_cuda.cuda.synchronize()
    assert np.array_equal(v["M"].cpu().numpy().view(np.uint32), M)
    assert np.array_equal(v["Phi"].cpu().numpy().view(np.uint64), Phi)
    s.status()


def test_large_batch_equals_single_renders(torch_cuda):
    """More than 2^19 pixels in all: 64 hit points a wave in the batch's range query."""
    work = [(scenes.box_scene(640, 500), 5000, 0.05), (scenes.box_scene(500, 431), 3000, 0.02)]
    b = api.Batch([w[0] for w in work], [api.sppm_params(w[1], r0=w[2], seed=5) for w in work])
    b.iterate(2)
    for im, (sc, n, r0) in zip(b.resolve(), work):
        s = api.Sppm(sc, api.sppm_params(n, r0=r0, seed=5))
        s.iterate(2)
        assert torch_cuda.equal(im, s.resolve())

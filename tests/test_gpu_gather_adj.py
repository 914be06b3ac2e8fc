"""The adjoint's range query with 4, 16 and 64 hit points a wave against the oracle's gradients.

The image sizes lie on both sides of 2^14 and 2^17 pixels, and the larger first
radius gives discs of hundreds of photons, which a whole wave scans.
"""
import numpy as np
import pytest

from paper_1505_06022_amd import api, scenes
from test_gpu_adjoint import _check_close

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    return torch


@pytest.mark.parametrize("width,height", [(37, 29), (128, 128), (129, 128), (512, 256), (513, 256)])
@pytest.mark.parametrize("r0", [0.01, 0.3])
def test_split_against_the_oracle(torch_cuda, oracle_lib, width, height, r0):
    torch = torch_cuda
    print("case: adjoint gather", width, height, r0, flush=True)
    sc = scenes.box_scene(width, height)
    mats = [m for m in range(len(sc.mat_rho)) if sc.mat_rho[m] > 0.0]
    g = torch.linspace(-1.0, 2.0, width * height, device="cuda")
    s = api.Sppm(sc, api.sppm_params(3001, r0=r0, seed=7, record_iterations=2))
    s.iterate(2)
    grad = s.adjoint(g, mats).cpu().numpy()
    s.destroy()
    ref, _ = oracle_lib.sppm_grad(oracle_lib.OracleScene(sc), 7, 3001, 2, g.cpu().numpy().astype(np.float64), mats,
                                  r0=r0)
    assert np.abs(ref).max() > 0.0
    _check_close(grad, ref)

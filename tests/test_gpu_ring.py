"""Iterations under way at once: three slots of hit points, photon stores and tables.

A handle that takes its stage times runs one iteration after another on one
slot; the pipelined handle has to give the same state, the same last photons
and hit points and the same gradients, bit for bit, whatever the lengths of its
calls, in the one-launch photon pass and in the two-launch one (beyond 2^18
paths), each with its share of the device.
"""
import numpy as np
import pytest

from paper_1505_06022_amd import api, scenes

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    return torch


@pytest.mark.parametrize("photons", [20_001, 270_001])
@pytest.mark.parametrize("gather", [api.GATHER_EXACT, api.GATHER_STOCHASTIC])
def test_calls_equal_the_serial_handle(torch_cuda, photons, gather):
    print("case: ring, photons", photons, "gather", gather, flush=True)
    sc = scenes.procedural_scene(width=160, height=91, hf_cells=60, sphere_level=3, glass_level=4, seed=11)
    bvh = api.build_bvh(sc.verts, sc.tri_mat)
    rec = 16 if gather == api.GATHER_EXACT else 0
    common = dict(r0=0.03, seed=3, gather_mode=gather, record_iterations=rec)
    serial = api.Sppm(sc, api.sppm_params(photons, profile=api.PROFILE_TIME, **common), bvh=bvh)
    ring = api.Sppm(sc, api.sppm_params(photons, **common), bvh=bvh)
    for n in (1, 2, 3, 4, 6):  # 16 iterations: every slot is first, last and in the middle of a call
        serial.iterate(n)
        ring.iterate(n)
        a, b = serial.views(), ring.views()
        torch_cuda.cuda.synchronize()
        for key in ("N", "R2", "tau", "D"):
            assert np.array_equal(a[key].cpu().numpy(), b[key].cpu().numpy()), (n, key)
        assert int(a["photon_count"].cpu()[0]) == int(b["photon_count"].cpu()[0]), n
        hit = a["hp_nrm"].cpu().numpy().view(np.int32)[:, 3] >= 0
        assert np.array_equal(a["hp_pos"].cpu().numpy()[hit], b["hp_pos"].cpu().numpy()[hit]), n
    assert torch_cuda.equal(serial.resolve(), ring.resolve())
    if rec:
        g = torch_cuda.linspace(-1.0, 2.0, 160 * 91, device="cuda")
        mats = [m for m in range(len(sc.mat_rho)) if sc.mat_rho[m] > 0.0]
        ga, gb = serial.adjoint(g, mats), ring.adjoint(g, mats)
        assert torch_cuda.equal(ga, gb) and float(ga.abs().max()) > 0.0

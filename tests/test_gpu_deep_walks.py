"""Chains of triangles whose rays need far more stack than the four-child walk has,
or with more levels than its nodes are built for, through every kernel that starts
a walk with one ray a lane: large batches, the two-batch launch, the renderer's
passes and a batch of scenes.  Compared with the binary walk bit for bit."""
import numpy as np
import pytest

from paper_1505_06022_amd import api, scenes
from test_gpu_wide import _chain, _wide_depth

pytestmark = pytest.mark.gpu
OPTS = dict(max_leaf=1, bins=2)
# triangles, ratio, largest: 20 to 32 levels (up to 95 stack entries of 24), and more than 32
CHAINS = [(280, 1.15, 1e9, (20, 32)), (500, 1.15, 1e12, (33, 99))]


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    return torch


def _rays(n, ratio, top, m, width):
    """Along +x past the first triangles: rays of all depths mixed in every wave."""
    rng = np.random.default_rng(m)
    rays = np.zeros((m, 8), np.float32)
    rays[:, 1:3] = rng.uniform(-0.3, 0.3, (m, 2)) * width
    rays[:, 4], rays[:, 7] = 1.0, np.inf
    rays[:, 5:7] = rng.uniform(-0.2, 0.2, (m, 2))
    rays[:, 3] = top * float(ratio) ** rng.integers(-n, 0, m)
    return rays


@pytest.mark.parametrize("n,ratio,top,levels", CHAINS)
@pytest.mark.parametrize("m", [65_537, 70_001])
def test_one_ray_a_lane(torch_cuda, oracle_lib, n, ratio, top, levels, m):
    verts = _chain(n, ratio, top)
    assert levels[0] <= _wide_depth(verts, **OPTS) <= levels[1]
    rays = _rays(n, ratio, top, m, float(verts[0].max()))
    bvh = api.build_bvh(verts, np.zeros(n, np.uint32), **OPTS)
    r = torch_cuda.from_numpy(rays).cuda()
    print("case: deep chain", n, "rays", m, flush=True)
    h0, t0 = api.trace_rays(bvh, r, kernel=api.TRACE_PER_RAY)
    hb, tb = oracle_lib.trace_brute_force(verts, rays[:2000])
    assert np.array_equal(h0[:2000].cpu().numpy(), hb) and np.array_equal(t0[:2000].cpu().numpy(), tb)
    assert len(torch_cuda.unique(h0)) > n // 4
    for kw in (dict(), dict(block=256), dict(kernel=api.TRACE_POSTPONED, refill=0),
               dict(kernel=api.TRACE_POSTPONED, refill=32, reorder=1, block=64),
               dict(kernel=api.TRACE_POSTPONED, refill=63, reorder=2)):
        h, t = api.trace_rays(bvh, r, **kw)
        assert torch_cuda.equal(h0, h) and torch_cuda.equal(t0, t), kw
    # one launch for a bucketed batch and an image in tiles: always one ray a lane
    w = 37
    k = m // w * w
    out = [torch_cuda.empty(s, dtype=d, device="cuda") for s, d in ((m, torch_cuda.int32), (m, torch_cuda.float32),
                                                                    (k, torch_cuda.int32), (k, torch_cuda.float32))]
    api.trace_rays_multi(bvh, [
        dict(rays=r, hit=out[0], t=out[1], kernel=api.TRACE_POSTPONED, refill=32, reorder=1, block=64),
        dict(rays=r[:k].contiguous(), hit=out[2], t=out[3], kernel=api.TRACE_PACKET, block=64, tile_width=w)])
    for got, ref in zip(out, (h0, t0, h0[:k], t0[:k])):
        assert torch_cuda.equal(got, ref)


def _scene(n, ratio, top):
    """The chain seen from its narrow end, with a light there that faces it."""
    box = scenes.box_scene(40, 30)
    light = int(np.argmax(box.mat_Le > 0))
    diffuse = int(np.argmax((box.mat_rho > 0) & (box.mat_Le == 0)))
    lamp = np.array([[[-1, -1, -1], [-1, 2, -1], [-1, -1, 2]]], np.float32)
    verts = np.concatenate([_chain(n, ratio, top), lamp]).astype(np.float32)
    mats = np.array([diffuse] * n + [light], np.uint32)
    cam = scenes.dataclasses.replace(box.camera, pos=(-1e-3, 0.0, 0.0), look=(1.0, 0.1, 0.1), up=(0.0, 1.0, 0.0))
    return scenes.dataclasses.replace(box, verts=verts, tri_mat=mats, camera=cam)


@pytest.mark.parametrize("n,ratio,top,levels", CHAINS)
@pytest.mark.parametrize("photons,kernel", [(5_001, 0), (270_001, 0), (5_001, 1), (5_001, 2), (5_001, 3)])
def test_renderer(torch_cuda, n, ratio, top, levels, photons, kernel):
    sc = _scene(n, ratio, top)
    assert levels[0] <= _wide_depth(sc.verts, **OPTS) <= levels[1]
    bvh = api.build_bvh(sc.verts, sc.tri_mat, **OPTS)
    print("case: renderer on a deep chain", n, "photons", photons, "kernel", kernel, flush=True)
    g = torch_cuda.linspace(-1.0, 2.0, 1200, device="cuda")
    out = []
    for single in (0, 1):
        s = api.Sppm(sc, api.sppm_params(photons, r0=top * 1e-3, seed=3, photon_kernel=kernel, record_iterations=3,
                                         single_link_set=single), bvh=bvh)
        s.iterate(3)
        s.status()
        v = s.views()
        out.append([v[k].clone() for k in ("hp_pos", "M", "N", "R2", "tau", "D")] +
                   [s.resolve(), s.adjoint(g, [int(sc.tri_mat[0])])])
        assert int(v["photon_count"][0]) > 0 and int((v["hp_nrm"].view(torch_cuda.int32)[:, 3] >= 0).sum()) > 600
        s.destroy()
    for a, b in zip(*out):
        assert torch_cuda.equal(a.view(-1).view(torch_cuda.uint8), b.view(-1).view(torch_cuda.uint8))


@pytest.mark.parametrize("n,ratio,top,levels", CHAINS)
def test_batch(torch_cuda, n, ratio, top, levels):
    """A scene of the batch on a chain; its own BVH is built inside, with larger leaves."""
    print("case: batch with a deep chain", n, flush=True)
    scs = [_scene(n, ratio, top), scenes.box_scene(48, 32)]
    images = []
    for single in (0, 1):
        prm = [api.sppm_params(5_001, r0=top * 1e-3, seed=3, single_link_set=single),
               api.sppm_params(3_001, r0=0.1, seed=4, single_link_set=single)]
        images.append(api.render_batch(scs, prm, 2, chunk=256))
    for a, b in zip(*images):
        assert torch_cuda.equal(a.view(torch_cuda.int32), b.view(torch_cuda.int32))

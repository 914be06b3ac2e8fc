"""Rays that miss the whole scene: the same answers as the binary walk where some,
all or none of a wave's rays do, and for whole batches of them no slower."""
import numpy as np
import pytest

from paper_1505_06022_amd import api, scenes

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    return torch


def _away(rays):
    out = rays.copy()
    out[:, :3] += 100.0
    out[:, 4:7] = np.abs(out[:, 4:7])
    return out


@pytest.mark.parametrize("tris", [1, 36, 5_000])
@pytest.mark.parametrize("n", [1_009, 70_003])
def test_hits(torch_cuda, tris, n):
    print("case: misses", tris, n, flush=True)
    sc = scenes.small_soup(tris, 6) if tris != 36 else scenes.box_scene()
    bvh = api.build_bvh(sc.verts, np.zeros(len(sc.verts), np.uint32))
    rays = scenes.random_rays(n, 8)
    miss = _away(rays)
    rng = np.random.default_rng(1)
    for which in (np.ones(n, bool), rng.random(n) < 0.5, rng.random(n) < 0.98, np.arange(n) // 64 % 2 == 0):
        r = torch_cuda.from_numpy(np.where(which[:, None], miss, rays)).cuda()
        ref = api.trace_rays(bvh, r, kernel=api.TRACE_PER_RAY)
        for kw in (dict(), dict(kernel=api.TRACE_POSTPONED, refill=16, reorder=1, block=64)):
            got = api.trace_rays(bvh, r, **kw)
            assert torch_cuda.equal(ref[0], got[0]) and torch_cuda.equal(ref[1], got[1]), kw
    assert which.any() and int((ref[0] >= 0).sum()) > 0 or tris == 1


def test_no_slower_than_the_binary_walk(torch_cuda):
    """2^23 rays, 61 and 64 us (89 before such waves ended at once)."""
    sc = scenes.procedural_scene(hf_cells=60, sphere_level=3, glass_level=4)
    bvh = api.build_bvh(sc.verts, sc.tri_mat)
    n = 1 << 23
    r = torch_cuda.from_numpy(_away(scenes.random_rays(n, 8))).cuda()
    h = torch_cuda.empty(n, dtype=torch_cuda.int32, device="cuda")
    t = torch_cuda.empty(n, device="cuda")
    e = [torch_cuda.cuda.Event(enable_timing=True) for _ in range(2)]
    times = {0: [], api.TRACE_PER_RAY: []}
    print("case: time of misses", flush=True)
    for _ in range(40):
        for kernel, ms in times.items():
            e[0].record()
            for _ in range(4):
                api.trace_rays(bvh, r, h, t, kernel=kernel)
            e[1].record()
            torch_cuda.cuda.synchronize()
            ms.append(e[0].elapsed_time(e[1]))
    assert int(h.max()) == -1
    assert np.median(times[0]) < 1.2 * np.median(times[api.TRACE_PER_RAY]), [np.median(v) for v in times.values()]

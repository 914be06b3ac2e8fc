"""A renderer that fits with two slots or one only, and rays through a BVH that
has no room for its four-child nodes, give what they give with all memory, bit
for bit.  In a process of its own, where device allocations above a limit fail."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu
HERE = os.path.dirname(os.path.abspath(__file__))

CODE = """
import ctypes, sys
sys.path.insert(0, {root!r})
shim = ctypes.CDLL({shim!r}, ctypes.RTLD_GLOBAL)
shim.malloc_limit.argtypes = [ctypes.c_size_t]
shim.malloc_fail.argtypes = [ctypes.c_long]
shim.malloc_largest.restype = ctypes.c_size_t
import torch
from paper_1505_06022_amd import api, scenes
sc = scenes.procedural_scene(width=160, height=91, hf_cells=60, sphere_level=3, glass_level=4, seed=11)
bvh = api.build_bvh(sc.verts, sc.tri_mat)
mats = [m for m in range(len(sc.mat_rho)) if sc.mat_rho[m] > 0.0]
g = torch.linspace(-1.0, 2.0, 160 * 91, device="cuda")
def render(**kw):
    s = api.Sppm(sc, api.sppm_params(r0=0.03, seed=3, **kw), bvh=bvh)
    for n in (1, 4, 2):
        s.iterate(n)
    out = [s.resolve()]
    if kw.get("record_iterations"):
        out.append(s.adjoint(g, mats))
    s.status()
    torch.cuda.synchronize()
    s.destroy()
    return out
for kw in (dict(n_photons=270_001, record_iterations=7), dict(n_photons=20_001, record_iterations=7),
           dict(n_photons=270_001, gather_mode=api.GATHER_STOCHASTIC),
           dict(n_photons=20_001, photon_kernel=api.PHOTON_REGEN)):
    print("case: fewer slots", kw, flush=True)
    shim.malloc_limit(1 << 62)
    ref = render(**kw)
    size = shim.malloc_largest()
    for slots in ((1,) if kw.get("photon_kernel") else (2, 1)):
        shim.malloc_limit(size - 1)
        got = render(**kw)
        assert 0 < shim.malloc_largest() < size
        size = shim.malloc_largest()
        assert all(torch.equal(a, b) for a, b in zip(ref, got)), (kw, slots)
    shim.malloc_limit(1 << 62)
rays = torch.from_numpy(scenes.random_rays(70_000, 4)).cuda()
soup = scenes.small_soup(40_000, 3)
# allocations of a build, in order: [scratch of the device build,] nodes and triangles, then the merge's scratch and
# the four-child nodes, which it can do without
for builder, must in ((api.BUILD_HOST_SAH, 2), (api.BUILD_GPU_LBVH, 3)):
    whole = api.trace_rays(api.build_bvh(soup.verts, soup.tri_mat, builder=builder), rays)
    for nth in range(must + 2):
        print("case: builder", builder, "allocation", nth, "fails", flush=True)
        shim.malloc_fail(nth)
        try:
            b = api.build_bvh(soup.verts, soup.tri_mat, builder=builder)
        except api.PMError as e:
            assert e.code == api.PM_ERR_NOMEM and nth < must, (nth, e)
            continue
        assert nth >= must, nth
        shim.malloc_fail(-1)
        got = api.trace_rays(b, rays)
        assert torch.equal(whole[0], got[0]) and torch.equal(whole[1], got[1]), nth
print("finished")
"""


def test_less_memory_same_results(tmp_path):
    shim = str(tmp_path / "libmalloc_limit.so")
    subprocess.run(["gcc", "-shared", "-fPIC", "-O1", os.path.join(HERE, "hip_malloc_limit.c"), "-o", shim, "-ldl"],
                   check=True)
    r = subprocess.run([sys.executable, "-u", "-c", CODE.format(root=os.path.dirname(HERE), shim=shim)],
                       capture_output=True, text=True, timeout=100)
    print(r.stdout)
    assert r.returncode == 0 and "finished" in r.stdout, r.stdout + r.stderr

"""What a call does when the device has no room for memory that it can do without.

On the CPU, with a stand-in for the HIP runtime whose device memory is set to
what is left.  A BVH does without its four-child nodes (the binary walks take
its rays), a renderer without the buffers of its scene fingerprint (the host
computes it), without a third slot and without a second, in this order.
"""
import numpy as np
import pytest

import fake_hip


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    return fake_hip.build(tmp_path_factory.mktemp("fake_hip"))


BVH = """
st = new_stream()
sc = scenes.small_soup({tris}, 3)
def build():
    return api.build_bvh(sc.verts, np.zeros(len(sc.verts), np.uint32), stream=st)
b = build()
info = b.info()
whole = used()  # without the scratch of the merge
b.destroy()
assert used() == 0
need = info["device_bytes"] + 256  # nodes and triangles, the pad node, the work counter
rays, hit, t = np.zeros((8, 8), np.float32), np.zeros(8, np.int32), np.zeros(8, np.float32)
for left in (need, need + 1000, whole, 1 << 40):
    memory(left)
    b = build()
    log()
    api._check(api.lib().pm_trace_rays(b.h, rays.ctypes.data, 8, hit.ctypes.data, t.ctypes.data, ctypes.c_void_p(st.cuda_stream)))
    names = [c[1] for c in log() if c[0] == "launch"]
    assert len(names) == 1 and "k_trace" in names[0], names
    assert ("k_trace_wide" in names[0]) == (left == 1 << 40), (left, names)
    b.destroy()
    assert used() == 0
memory(need // 2)
try:
    build()
    assert False
except api.PMError as e:
    assert e.code == api.PM_ERR_NOMEM
assert used() == 0
print("ok")
"""


@pytest.mark.parametrize("tris", [20_000, 60_000])
def test_bvh_without_room_for_the_wide_nodes(lib, tris):
    assert "ok" in fake_hip.run(lib, BVH.format(tris=tris))


RENDERER = """
import struct
st = new_stream()
sc = scenes.small_soup(40_000, 3)
sc.camera = scenes.dataclasses.replace(sc.camera, width=64, height=48)
b = api.build_bvh(sc.verts, sc.tri_mat, stream=st)
base = used()
def make():
    log()
    s = api.Sppm(sc, api.sppm_params(1 << 14), bvh=b, stream=st)
    return s, [int(c[1]) for c in log() if c[0] == "malloc"]
s, sizes = make()
hash_bytes, three = sizes
s.destroy()
def fingerprint(s):
    n = ctypes.c_uint64(0)
    api._check(api.lib().pm_sppm_save(s.h, None, ctypes.byref(n), None))
    buf = ctypes.create_string_buffer(n.value)
    api._check(api.lib().pm_sppm_save(s.h, buf, ctypes.byref(n), ctypes.c_void_p(st.cuda_stream)))
    return struct.unpack_from("<Q", buf.raw, 40)[0]
h, words = 0xcbf29ce484222325, []
cam = sc.camera
for a in (np.array([len(sc.verts)], np.int64), sc.verts, sc.tri_mat, np.array([len(sc.mat_type)], np.int32), sc.mat_type,
          sc.mat_rho, sc.mat_q, sc.mat_Le, sc.mat_ior, np.array(cam.pos + cam.look + cam.up + (cam.tan_half_fov,), np.float32),
          np.array([cam.width, cam.height], np.int32)):
    words += np.ascontiguousarray(a).ravel().view(np.uint32).tolist()
for w in words:
    h = (h ^ w) * 0x100000001b3 & 0xffffffffffffffff
# no room for the fingerprint's words: the host hashes them
fail("hipMalloc", 0, OOM)
s, sizes = make()
assert sizes == [three], sizes
assert fingerprint(s) == h
s.iterate(4, stream=st)
s.destroy()
# room for either: the words first, then the whole handle
memory(base + three)
s, sizes = make()
assert sizes[-1] == three, sizes
s.destroy()
# fewer slots: the photon passes of two iterations at once, then of one
limit = three - 1
for streams in (2, 1):
    memory(base + limit)
    s, sizes = make()
    assert sizes[-1] <= limit
    limit = sizes[-1] - 1
    s.iterate(5, stream=st)
    calls = log()
    assert not unjoined(calls, st.cuda_stream)
    assert len(set(c[-1] for c in calls if c[0] == "launch" and "k_photon" in c[1])) == streams
    s.destroy()
memory(base + limit)
try:
    make()
    assert False
except api.PMError as e:
    assert e.code == api.PM_ERR_NOMEM, e
assert used() == base
print("ok")
"""


def test_renderer_in_little_memory(lib):
    assert "ok" in fake_hip.run(lib, RENDERER)

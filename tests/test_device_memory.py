"""What a call does when the device has no room for memory that it can do without.

On the CPU, with a stand-in for the HIP runtime whose device memory is set to
what is left.  A BVH does without its four-child nodes: the binary walks take
its rays.
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

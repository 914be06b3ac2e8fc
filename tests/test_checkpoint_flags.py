"""A checkpoint keeps the overflow flag of every slot, read once the copy from the
device has ended.  On the CPU, with a stand-in for the HIP runtime that copies to
the host as late as the runtime may."""
import pytest

import fake_hip


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    return fake_hip.build(tmp_path_factory.mktemp("fake_hip"))


CODE = """
st = new_stream()
sc = scenes.box_scene(16, 16)
bvh = api.build_bvh(sc.verts, sc.tri_mat, stream=st)
def handle():
    return api.Sppm(sc, api.sppm_params(1 << 10), bvh=bvh, stream=st)
def counters(s):
    v = api.SppmViews()
    v.size = ctypes.sizeof(api.SppmViews)
    api._check(api.lib().pm_sppm_get_views(s.h, ctypes.byref(v)))
    return np.ctypeslib.as_array(ctypes.cast(v.photon_count, ctypes.POINTER(ctypes.c_uint32)), (4,))
def status(s):
    try:
        s.status(stream=st)
        return 0
    except api.PMError as e:
        return e.code
for k in (1, 2, 3, 4):  # the slot of the last iteration: 0, 1, 2, 0
    for flag in (0, 1, 2):
        a, b = handle(), handle()
        a.iterate(k, stream=st)
        counters(a)[1] = flag
        assert (status(a) == api.PM_ERR_OVERFLOW) == (flag != 0), (k, flag)
        b.load(a.save(stream=st), stream=st)
        assert status(b) == status(a), (k, flag)
        a.destroy()
        b.destroy()
print("ok")
"""


def test_flags_of_all_slots(lib):
    assert "ok" in fake_hip.run(lib, CODE)

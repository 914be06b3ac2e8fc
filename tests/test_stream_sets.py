"""The streams that released renderers leave for the next ones: bounded, used by
one renderer at a time, and not used again once a device reset has ended them.  On
the CPU, with a stand-in for the HIP runtime."""
import pytest

import fake_hip


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    return fake_hip.build(tmp_path_factory.mktemp("fake_hip"))


CODE = """
st = new_stream()
sc = scenes.box_scene(16, 16)
prm = api.sppm_params(1 << 10)
def streams(calls):
    return [c[1] for c in calls if c[0] == "stream+"], [c[1] for c in calls if c[0] == "stream-"]
def use(s):
    log()
    s.iterate(4, stream=st)
    calls = log()
    assert not unjoined(calls, st.cuda_stream)
    return {c[-1] for c in calls if c[0] == "launch"}
bvh = api.build_bvh(sc.verts, sc.tri_mat, stream=st)
log()
six = [api.Sppm(sc, prm, bvh=bvh, stream=st) for _ in range(6)]
made, gone = streams(log())
assert len(made) - len(gone) == 4 * 6
used_by = [use(s) for s in six]
assert len(set().union(*used_by)) == sum(map(len, used_by))  # no two share a stream
for s in six:
    s.destroy()
assert len(streams(log())[1]) == 4 * 2  # four sets stay
s = api.Sppm(sc, prm, bvh=bvh, stream=st)
assert streams(log()) == ([], []) and use(s) <= set().union(*used_by)
s.destroy()
fake.fake_device_reset()
st = new_stream()
bvh = api.build_bvh(sc.verts, sc.tri_mat, stream=st)
log()
s = api.Sppm(sc, prm, bvh=bvh, stream=st)
assert len(streams(log())[0]) == 7
use(s)
s.destroy()
print("ok")
"""


def test_kept_sets(lib):
    assert "ok" in fake_hip.run(lib, CODE)

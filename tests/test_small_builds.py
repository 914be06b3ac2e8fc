"""A small tree's build makes few device calls: one allocation, no kernel, one
wait.  On the CPU, with a stand-in for the HIP runtime, whose device memory also
shows that nodes and triangles arrive where they are read."""
import pytest

import fake_hip


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    return fake_hip.build(tmp_path_factory.mktemp("fake_hip"))


CODE = """
st = new_stream()
v = scenes.small_soup({tris}, 2).verts
nodes, tris, info = api.build_bvh_host(v, None)
small = info["n_nodes"] <= 8192
log()
b = api.build_bvh(v, None, stream=st)
calls = log()
count = lambda word: sum(c[0] == word for c in calls)
if small:
    assert count("malloc") == 1 and count("launch") == 0 and count("sync") == 1 and count("fill") == 0, calls
    assert count("copy") == (1 if info["device_bytes"] < 100_000 else 3), calls
else:
    assert count("launch") > 0
got = b.download(stream=st)
assert np.array_equal(got[0].reshape(-1), nodes.reshape(-1)) and np.array_equal(got[1].reshape(-1), tris.reshape(-1))
b.destroy()
assert used() == 0
print("ok", info["n_nodes"])
"""


@pytest.mark.parametrize("tris", [1, 2, 36, 400, 2_000, 8_200, 8_600])
def test_calls_of_a_build(lib, tris):
    assert "ok" in fake_hip.run(lib, CODE.format(tris=tris))

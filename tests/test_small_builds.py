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


# The four-child nodes of a small tree, in their place after the nodes: from the root down a node takes a binary node's
# children and opens the inner one of largest area until it has four; they are numbered in the binary nodes' order.
NODES = """
st = new_stream()
v = scenes.small_soup({tris}, {seed}).verts
nodes, _, info = api.build_bvh_host(v, None, max_leaf={leaf})
q, step, n = nodes[0], np.asarray(info["grid_step"], np.float32), info["n_nodes"]
log()
b = api.build_bvh(v, None, max_leaf={leaf}, stream=st)
leaf = lambda w: w >> 31 != 0
def area(k):
    x, y, z = [np.float32((int(q[k, a]) >> 16) - (int(q[k, a]) & 0xffff)) * step[a] for a in range(3)]
    return (x * y + y * z) + z * x
def kids(k):
    if leaf(q[k, 3]):
        return [k]
    out, at = [k], 0
    while len(out) < 4:
        k = out[at]
        out[at] = k + 1
        out.append(k + 2 if leaf(q[k + 1, 3]) else int(q[k + 1, 3]))
        inner = [i for i in range(len(out)) if not leaf(q[out[i], 3])]
        if not inner:
            break
        at = max(inner, key=lambda i: (area(out[i]), -i))
    return out
wide, todo = dict(), [0]
while todo:
    k = todo.pop()
    wide[k] = kids(k)
    todo += [c for c in wide[k] if not leaf(q[c, 3]) and c != k]
number = dict((k, i) for i, k in enumerate(sorted(wide)))
want = np.zeros((len(wide), 4, 4), np.uint32)
want[:] = (0xffff, 0xffff, 0xffff, 0x80000000)
for k, cs in wide.items():
    for i, c in enumerate(cs):
        want[number[k], i] = q[c]
        if not leaf(q[c, 3]):
            want[number[k], i, 3] = number[c]
at = (6 * 16 * n + 16 + 255) // 256 * 256
got = np.ctypeslib.as_array(ctypes.cast(fake.fake_last_block() + at, ctypes.POINTER(ctypes.c_uint32)), (want.size,))
assert np.array_equal(got, want.reshape(-1))
print("ok", len(wide))
"""


@pytest.mark.parametrize("tris,leaf,seed", [(1, 4, 1), (2, 1, 1), (5, 1, 3), (7, 7, 3), (36, 4, 5), (300, 1, 2), (2_000, 4, 7)])
def test_four_child_nodes(lib, tris, leaf, seed):
    assert "ok" in fake_hip.run(lib, NODES.format(tris=tris, leaf=leaf, seed=seed))

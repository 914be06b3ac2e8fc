"""Handles and batches whose rays take only the binary walk launch kernels without
the other walk's stacks, and their photon passes take the device they need.

On the CPU: the kernels that a stand-in for the HIP runtime is asked to launch,
and the LDS that the built library reserves for them.
"""
import json

import pytest

import fake_hip
from paper_1505_06022_amd import build

STACK = 64 * 24 * 4  # bytes of LDS a wave for the four-child walk
SINK = 2 * 112 * 16  # and for its photons on their way to the store


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    return fake_hip.build(tmp_path_factory.mktemp("fake_hip"))


@pytest.fixture(scope="module")
def lds():
    return {k: v[".group_segment_fixed_size"] for k, v in fake_hip.kernels(build.OUT).items()}


CODE = """
import json
st = new_stream()
sc = scenes.box_scene(16, 16)
verts = np.concatenate([scenes.small_soup(9000, 2).verts, sc.verts]).astype(np.float32)
sc = scenes.dataclasses.replace(sc, verts=verts, tri_mat=np.concatenate([np.zeros(9000, np.uint32), sc.tri_mat]))
if {without_nodes}:
    fail("hipMalloc", 2, OOM)  # the scratch that the nodes are merged in
bvh = api.build_bvh(sc.verts, sc.tri_mat, stream=st)
out = dict()
for name, kw in {cases}.items():
    s = api.Sppm(sc, api.sppm_params(store_factor=1, **kw), bvh=bvh, stream=st)
    log()
    s.iterate(2, stream=st)
    if kw.get("record_iterations"):
        g, grad, mats = np.zeros(256, np.float32), np.zeros(2), np.zeros(1, np.int32)
        api._check(api.lib().pm_sppm_adjoint(s.h, g.ctypes.data, mats.ctypes.data, 1, grad.ctypes.data,
                                             ctypes.c_void_p(st.cuda_stream)))
    out[name] = [(c[1], int(c[2])) for c in log() if c[0] == "launch" and ("k_eye" in c[1] or "k_photon" in c[1])]
    s.destroy()
print(json.dumps(out))
"""
KERNELS = {"auto": "n_photons=1 << 20, record_iterations=2", "few": "n_photons=1 << 12, record_iterations=2",
           "stochastic": "n_photons=1 << 20, gather_mode=1", **{f"kernel{k}": f"n_photons=1 << 20, photon_kernel={k}"
                                                               for k in (1, 2, 3, 6)}}


def _launches(lib, more="", without_nodes=False):
    cases = "{" + ", ".join(f"{n!r}: dict({kw}{more})" for n, kw in KERNELS.items()) + "}"
    return json.loads(fake_hip.run(lib, CODE.format(cases=cases, without_nodes=without_nodes)).splitlines()[-1])


@pytest.mark.parametrize("why", ["one link set", "no four-child nodes"])
def test_binary_walk_kernels_have_no_stacks(lib, lds, why):
    wide = _launches(lib)
    binary = _launches(lib, ", single_link_set=3") if why == "one link set" else _launches(lib, without_nodes=True)
    for name in KERNELS:
        assert any(lds[k] >= 4 * STACK for k, _ in wide[name]), name
        assert len(binary[name]) == len(wide[name])
        for k, _ in binary[name]:
            assert lds[k] <= (0 if "k_eye" in k else 4 * SINK), (name, k)
    # the binary walk's passes take twice the share (see shares_of)
    for part, share in (("k_photon_head", 1), ("k_photon_tail", 2)):
        grid = {g for k, g in binary["auto"] if part in k}
        assert grid == {256 * 4 // share}, (part, grid)
        assert {g for k, g in wide["auto"] if part in k} == {256 * 4 // share // 2}


BATCH = """
import json
st = new_stream()
out = dict()
for name, sets in dict(wide=(0, 0), mixed=(0, 2), binary=(1, 6)).items():
    scs = [scenes.box_scene(16, 16), scenes.box_scene(24, 16)]
    prm = [api.sppm_params(1 << 12, single_link_set=k) for k in sets]
    b = api.Batch(scs, prm, stream=st, {opts})
    b.iterate(1, stream=st)
    out[name] = [c[1] for c in log() if c[0] == "launch" and "k_batchILi" in c[1]]
    b.destroy()
print(json.dumps(out))
"""


@pytest.mark.parametrize("opts", ["block=128", "block=256", "block=256, use_graph=False"])
def test_batch_of_binary_walks_has_no_stacks(lib, lds, opts):
    out = json.loads(fake_hip.run(lib, BATCH.format(opts=opts)).splitlines()[-1])
    waves = 2 if "128" in opts else 4
    for name, kernels in out.items():
        assert len(kernels) == 7
        most = max(lds[k] for k in kernels)
        assert most >= waves * STACK if name != "binary" else most <= waves * SINK + 4, (name, most)

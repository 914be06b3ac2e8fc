"""A cached autotuner result holds for the item rules that it was measured under:
an entry in the form written before they changed is not used.  On the CPU, with a
stand-in for the HIP runtime (every candidate takes the same time there)."""
import pytest

import fake_hip


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    return fake_hip.build(tmp_path_factory.mktemp("fake_hip"))


CODE = """
import os
path = {path!r}
os.environ["PM_AUTOTUNE_CACHE"] = path
st = new_stream()
scs = [scenes.box_scene(16, 16), scenes.box_scene(24, 16)]
prm = [api.sppm_params(1 << 10), api.sppm_params(1 << 11)]
text = "fake:2" + "".join(f":{{s.camera.width * s.camera.height}},{{p.n_photons}},{{len(s.verts)}}" for s, p in zip(scs, prm))
h = 1469598103934665603
for c in text.encode():
    h = (h ^ c) * 1099511628211 & 0xffffffffffffffff
open(path, "w").write(f"{{h:016x}} 64 128 0.001\\n")
def info(**kw):
    b = api.Batch(scs, prm, autotune=True, stream=st, **kw)
    i = b.info()
    b.destroy()
    return i
i = info()
assert not i["tuned_from_cache"] and len(i["candidates"]) == 8, i
assert info()["tuned_from_cache"]  # its own entry is
prm = [api.sppm_params(1 << 10, single_link_set=1), api.sppm_params(1 << 11, single_link_set=2)]
assert not info()["tuned_from_cache"]  # measured for the other walk
print("ok")
"""


def test_entry_of_other_rules(lib, tmp_path):
    assert "ok" in fake_hip.run(lib, CODE.format(path=str(tmp_path / "tune.txt")))

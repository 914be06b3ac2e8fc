"""A build refused for a non-finite vertex has made no device call: nothing is
allocated or enqueued, so a recording on the stream goes on.  On the CPU, with a
stand-in for the HIP runtime; the places are those where the check's runs of
4,096 values and its threads' parts (of 2^21 values at least) begin and end."""
import pytest

import fake_hip


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    return fake_hip.build(tmp_path_factory.mktemp("fake_hip"))


CODE = """
st = new_stream()
log()
def build(v):
    try:
        api.build_bvh(v, None, builder={builder}, stream=st).destroy()
        return 0, ""
    except api.PMError as e:
        return e.code, str(e)
n = 1000
good = np.full((n, 3, 3), np.finfo(np.float32).max, np.float32)
good[::2] = -good[::2]
good[1::3] = 1e-40  # subnormal
for bad in (np.inf, -np.inf, np.nan, -np.nan):
    for at in (0, 8, 9, 4095, 4096, 8191, 8192, 9 * n - 1):
        v = good.copy()
        v.reshape(-1)[at] = bad
        v.reshape(-1)[9 * n - 1] = bad
        fake.fake_capture(st.cuda_stream, 1)
        code, text = build(v)
        fake.fake_capture(st.cuda_stream, 0)
        assert code == api.PM_ERR_ARG and text.endswith(f"triangle {{at // 9}}"), (bad, at, text)
        assert log() == [], (bad, at)
code, text = build(good)  # finite: the build begins
assert log() and "non-finite" not in text
fail("hipMalloc", 0, OOM)  # an error of the runtime stays one
assert build(good)[0] == api.PM_ERR_NOMEM
print("ok")
"""


@pytest.mark.parametrize("builder", ["api.BUILD_HOST_SAH", "api.BUILD_GPU_LBVH"])
def test_nothing_enqueued(lib, builder):
    assert "ok" in fake_hip.run(lib, CODE.format(builder=builder))


PARTS = """
st = new_stream()
log()
n = 9 * 700_001
v = np.random.default_rng(1).uniform(-1, 1, n).astype(np.float32)
part = (n // 3 + 4095) // 4096 * 4096
for first in (0, part - 1, part, part + 1, 2 * part - 1, 2 * part, n - 2, n - 1):
    for second in (first, n - 1):
        bad = v.copy()
        bad[first] = np.nan
        bad[second] = np.inf
        try:
            api.build_bvh(bad.reshape(-1, 3, 3), None, builder=api.BUILD_GPU_LBVH, stream=st)
            assert False
        except api.PMError as e:
            assert e.code == api.PM_ERR_ARG and str(e).endswith(f"triangle {first // 9}"), (first, second, e)
assert log() == []
print("ok")
"""


def test_first_of_several_parts(lib):
    assert "ok" in fake_hip.run(lib, PARTS)

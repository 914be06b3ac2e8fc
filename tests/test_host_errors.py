"""A call that fails on the way leaves no work that its caller's stream does not wait for,
and no error for the next call to report.

On the CPU, with a stand-in for the HIP runtime: each runtime call that an
iteration or an adjoint makes fails once, and the streams and events that the
call used are followed.
"""
import pytest

import fake_hip


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    return fake_hip.build(tmp_path_factory.mktemp("fake_hip"))


HANDLES = {
    "two_phase": "dict(n_photons=1 << 20, store_factor=1)",
    "one_launch": "dict(n_photons=1 << 12)",
    "regen": "dict(n_photons=1 << 12, photon_kernel=api.PHOTON_REGEN)",
    "serial": "dict(n_photons=1 << 12, profile=api.PROFILE_TIME)",
    "stochastic": "dict(n_photons=1 << 12, gather_mode=api.GATHER_STOCHASTIC)",
}

CODE = """
kw = {kw}
recorded = kw.get("gather_mode", 0) == 0
if recorded:
    kw["record_iterations"] = 5
st = new_stream()
sc = scenes.box_scene(16, 16)
bvh = api.build_bvh(sc.verts, sc.tri_mat, stream=st)
s = api.Sppm(sc, api.sppm_params(**kw), bvh=bvh, stream=st)
image_grad, grad, mats = np.zeros(256, np.float32), np.zeros(2), np.zeros(1, np.int32)
def iterate():
    s.iterate(5, stream=st)
def adjoint():
    api._check(api.lib().pm_sppm_adjoint(s.h, image_grad.ctypes.data, mats.ctypes.data, 1, grad.ctypes.data,
                                         ctypes.c_void_p(st.cuda_stream)))
def sweep(call):
    log()
    call()
    calls = log()
    assert not unjoined(calls, st.cuda_stream)
    for what, word in (("hipLaunchKernel", "launch"), ("hipEventRecord", "record"), ("hipStreamWaitEvent", "wait")):
        total = sum(c[0] == word for c in calls)
        assert total > 4
        for nth in range(total):
            fail(what, nth, INVALID)
            try:
                call()
                assert False, ("no error", what, nth)
            except api.PMError as e:
                assert e.code == api.PM_ERR_HIP
            loose = unjoined(log(), st.cuda_stream)
            assert not loose, (call.__name__, what, nth, loose)
            assert fake.hipGetLastError() == 0, (call.__name__, what, nth)
iterate()
if recorded:
    sweep(adjoint)
sweep(iterate)
print("ok")
"""


@pytest.mark.parametrize("handle", HANDLES)
def test_failed_calls_leave_no_loose_work(lib, handle):
    assert "ok" in fake_hip.run(lib, CODE.format(kw=HANDLES[handle]))

"""What overlapped iterations may not overtake, with three slots and with two: every
writer of a slot comes after the slot's readers of `ring` iterations ago, every
reader after its writers.  On the CPU, with a stand-in for the HIP runtime: the
launches of a call with the streams and events that order them."""
import pytest

import fake_hip


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    return fake_hip.build(tmp_path_factory.mktemp("fake_hip"))


CODE = """
kw, slots = {kw}, {slots}
st = new_stream()
sc = scenes.box_scene(16, 16)
bvh = api.build_bvh(sc.verts, sc.tri_mat, stream=st)
exact = not kw.get("gather_mode")
prm = api.sppm_params(store_factor=1, record_iterations=64 if exact else 0, **kw)

def launches(calls):
    # each launch with the work of every stream that it follows (its own included)
    follows, events, out = dict(), dict(), []
    for c in calls:
        if c[0] == "launch":
            mine = follows.setdefault(c[-1], dict())
            mine[c[-1]] = mine.get(c[-1], 0) + 1
            out.append((c[1], c[-1], dict(mine)))
        elif c[0] == "record":
            events[c[1]] = dict(follows.get(c[2], dict()))
        elif c[0] == "wait":
            mine = follows.setdefault(c[1], dict())
            for s, n in events.get(c[2], dict()).items():
                mine[s] = max(mine.get(s, 0), n)
    return out

def check(n, adjoint):
    all_ = launches(log())
    def of(*names):
        found = [x for x in all_ if any(m in x[0] for m in names)]
        assert len(found) == n, (names, len(found), n)
        return found
    def ordered(a, b, what):
        assert b[2].get(a[1], 0) >= a[2][a[1]], (what, a[0], b[0], adjoint, n)
    photon_first, eye = of("k_photon_begin"), of("k_eye")
    photon_last = of("k_adj_phimax") if adjoint else of(*[k for k in ("k_photon_tail", "k_photon_regen", "k_photonI", "k_photon_stream",
                                                                     "k_photon_pool", "k_photon_drain") if any(k in x[0] for x in all_)])
    grid = of("k_count") if exact else of("k_sh_insert")
    store_read = of("k_path_adj") if adjoint else of("k_scatter") if exact else of("k_sh_gather")
    query = of("k_gather_adj") if adjoint else of("k_gatherI") if exact else of("k_sh_gather")
    hits_read, clear, rmax = (query if adjoint else of("k_update")), of("k_rmax_clear"), of("k_rmaxE")
    for k in range(n):
        for a, b in ((photon_last, grid), (eye, rmax), (clear, rmax), (rmax, grid)):
            ordered(a[k], b[k], k)
        if adjoint:
            ordered(photon_last[k], of("k_adj_scale")[k], k)
            ordered(of("k_adj_gmax")[k], of("k_adj_scale")[k], k)
        if k + slots < n:
            for a, b in ((store_read, photon_first), (hits_read, eye), (query, clear)):
                ordered(a[k], b[k + slots], ("slot", k))
        if k + 1 < n:
            ordered(store_read[k], grid[k + 1], k)
            if not adjoint:
                ordered(hits_read[k], rmax[k + 1], k)
    # and iterations do overlap
    assert n == 1 or any(photon_first[k + 1][2].get(store_read[k][1], 0) < store_read[k][2][store_read[k][1]] for k in range(n - 1))

log()
s = api.Sppm(sc, prm, bvh=bvh, stream=st)
size = max(int(c[1]) for c in log() if c[0] == "malloc")
if slots < {most}:
    s.destroy()
    memory(used() + size - 1)
    s = api.Sppm(sc, prm, bvh=bvh, stream=st)
for capture in (0, 1):
    fake.fake_capture(st.cuda_stream, capture)
    for n in (1, 2, 3, 7):
        log()
        s.iterate(n, stream=st)
        check(n, False)
    if exact:
        g, grad, mats = np.zeros(256, np.float32), np.zeros(2), np.zeros(1, np.int32)
        log()
        api._check(api.lib().pm_sppm_adjoint(s.h, g.ctypes.data, mats.ctypes.data, 1, grad.ctypes.data,
                                             ctypes.c_void_p(st.cuda_stream)))
        check(13 * (1 + capture), True)
print("ok")
"""


@pytest.mark.parametrize("kw,most", [("dict(n_photons=1 << 20)", 3), ("dict(n_photons=1 << 12)", 3),
                                     ("dict(n_photons=1 << 20, single_link_set=2)", 3),
                                     ("dict(n_photons=1 << 20, gather_mode=api.GATHER_STOCHASTIC)", 3)] +
                         [(f"dict(n_photons=1 << 12, photon_kernel={k})", 3 if k == 6 else 2) for k in range(1, 7)])
def test_order(lib, kw, most):
    for slots in range(2, most + 1):
        assert "ok" in fake_hip.run(lib, CODE.format(kw=kw, slots=slots, most=most))

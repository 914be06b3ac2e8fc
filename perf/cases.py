"""Workloads of the photon-mapping library, each one pass through its public entry points.

A case is a dict of plain values.  `listed()` names the fixed ones, `draw(rng)`
gives another of the same ranges, `prepare` builds what a program holds before
the call (scene, rays, BVH, renderer handle), `run` makes the call, `work` gives
the bytes and operations no implementation can do without, and `exact` the
closest-hit distances in 64-bit arithmetic where brute force is affordable.

Kinds:
  trace    closest hits of ray batches against a prepared BVH.  call "default"
           (no options), "bucketed" (the options for incoherent batches),
           "noalloc" (the same on the static scratch, for callers that must not
           allocate), or "pair" (a camera batch as packets over pixel tiles and
           an incoherent batch in one call).
  rebuild  a deforming scene's frame: the BVH built on the device from host
           vertices, then its primary rays.
  sppm     a progressive renderer that is kept: `iters` more iterations and the
           image so far.
  render   one whole render in one call, from scene description to image.
  diff     one optimisation step on the albedos and the light: differentiable
           render, L2 loss against a target, gradients.
  batch    several renderers of uneven size advanced together.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1505_06022_amd import api, scenes

# Options for incoherent and for camera batches: those of the benchmark's timed call.
INCOHERENT = dict(kernel=api.TRACE_POSTPONED, refill=32, reorder=1, block=64)
CAMERA = dict(kernel=api.TRACE_PACKET, block=64)


def _trace(name, scene, tris, call, width=0, height=0, rays=0, split=False):
    return dict(name=name, kind="trace", scene=scene, tris=tris, call=call, width=width, height=height, rays=rays,
                split=split)


def _light(kind, name, cells, sphere, glass, width, height, photons, iters, **more):
    return dict(name=name, kind=kind, scene="procedural", cells=cells, sphere=sphere, glass=glass, width=width,
                height=height, photons=photons, iters=iters, **more)


def listed():
    return [
        # A picking or visibility query: a thousand rays into a 36-triangle room; launches and latency.
        _trace("trace_box_1009", "box", 36, "default", rays=1009),
        # The primary rays of a frame of the 250k-triangle scene, traced with no options.
        _trace("trace_camera_procedural", "procedural", 250_094, "default", width=1280, height=720),
        # A ragged incoherent batch (one bounce of a path tracer) on a mid-size soup with the default build.
        _trace("trace_incoherent_odd", "soup", 1 << 18, "bucketed", rays=300_007),
        # The traversal workload of the benchmark: 2^20 triangles, 1920x1080 camera rays and 2^21 incoherent rays.
        _trace("trace_pair_soup", "soup", 1 << 20, "pair", width=1920, height=1080, rays=1 << 21, split=True),
        # Geometry that changes every frame: device BVH build and a 640x360 preview's primary rays.
        dict(name="rebuild_soup", kind="rebuild", tris=131_072, width=640, height=360),
        # The small box scene of the tests, progressive preview: two iterations and the image.
        dict(name="sppm_box", kind="sppm", scene="box", width=64, height=64, photons=1 << 14, iters=2, gather=0),
        # The benchmark's SPPM workload: 250k triangles, 1280x720, 2^20 photons per iteration.
        _light("sppm", "sppm_procedural", 231, 5, 6, 1280, 720, 1 << 20, 8, gather=0),
        # The stochastic spatial hashing estimator on a quarter-size image.
        _light("sppm", "sppm_stochastic", 100, 4, 5, 640, 360, 1 << 18, 4, gather=1),
        # A thumbnail in one call: odd image and photon counts, handle creation and release included.
        _light("render", "render_thumbnail", 60, 3, 4, 333, 187, 100_003, 8),
        # One gradient step at the size used to check gradients.
        _light("diff", "diff_step_small", 231, 5, 6, 320, 180, 1 << 16, 4),
        # One gradient step at the benchmark's size.
        _light("diff", "diff_step_full", 231, 5, 6, 1280, 720, 1 << 20, 8),
        # Uneven scenes rendered together, as for a data set of small images.
        dict(name="batch_uneven", kind="batch", scenes=8, tri_hi=50_000, side_hi=320, log2_photons_hi=18, iters=2),
    ]


def _log_int(rng, lo, hi):
    """An integer log-uniform in [lo, hi], odd half of the time."""
    v = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    return max(lo, min(hi, v | 1 if rng.random() < 0.5 else v))


def draw(rng):
    kind = rng.choice(["trace", "trace", "trace", "rebuild", "sppm", "sppm", "render", "diff", "batch"])
    if kind == "trace":
        call = rng.choice(["default", "default", "bucketed", "noalloc", "pair"])
        scene = "soup" if call != "default" else rng.choice(["soup", "procedural", "box"])
        tris = 36 if scene == "box" else 250_094 if scene == "procedural" else _log_int(rng, 1 << 10, 1 << 19)
        image = call == "pair" or (call == "default" and rng.random() < 0.5)
        width = _log_int(rng, 64, 1920) if image else 0
        height = max(1, int(width * rng.uniform(0.4, 0.8))) if image else 0
        rays = 0 if image and call != "pair" else _log_int(rng, 1000, 1 << 21)
        case = _trace("", scene, tris, call, width, height, rays, split=scene == "soup" and rng.random() < 0.3)
    elif kind == "rebuild":
        width = _log_int(rng, 160, 1280)
        case = dict(kind="rebuild", tris=_log_int(rng, 1 << 10, 1 << 19), width=width, height=width * 9 // 16 + 1)
    elif kind == "batch":
        case = dict(kind="batch", scenes=rng.randint(2, 10), tri_hi=_log_int(rng, 5_000, 50_000),
                    side_hi=_log_int(rng, 140, 320), log2_photons_hi=rng.choice([17, 18]), iters=rng.randint(1, 3))
    else:
        width = _log_int(rng, 48, 960)
        height = max(16, int(width * rng.uniform(0.4, 1.0)))
        cells, sphere = _log_int(rng, 12, 231), rng.randint(1, 5)
        photons = _log_int(rng, 1 << 12, 1 << 19)
        iters = rng.randint(2, 8) if kind != "diff" else rng.randint(2, 6)
        case = _light(kind, "", cells, sphere, min(6, sphere + 1), width, height, photons, iters)
        if kind == "sppm":
            case["gather"] = 1 if rng.random() < 0.25 else 0
    case.pop("name", None)
    return case


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------
def _scene(case, seed):
    if case.get("scene") == "box":
        return scenes.box_scene(case.get("width") or 64, case.get("height") or 64)
    if case.get("scene") == "procedural":
        return scenes.procedural_scene(width=case["width"] or 64, height=case["height"] or 64,
                                       hf_cells=case.get("cells", 231), sphere_level=case.get("sphere", 5),
                                       glass_level=case.get("glass", 6), seed=seed)
    return scenes.soup_scene(case["tris"], seed)


def _camera_rays(scene, width, height):
    cam = scenes.dataclasses.replace(scene.camera, width=width, height=height)
    return torch.from_numpy(scenes.pinhole_rays(cam)).cuda()


def _r0(scene, width):
    v = scene.verts.reshape(-1, 3)
    return 0.05 * float(np.linalg.norm(v.max(0) - v.min(0))) * 64 / width


def _params(case, scene, seed, **more):
    return api.sppm_params(case["photons"], alpha=0.7, r0=_r0(scene, case["width"]), seed=seed, **more)


def _rays(case, scene, seed):
    """(camera rays or None, incoherent rays or None) as host arrays."""
    cam = inc = None
    if case["width"]:
        c = scenes.dataclasses.replace(scene.camera, width=case["width"], height=case["height"])
        cam = scenes.pinhole_rays(c)
    if case["rays"]:
        inc = scenes.random_rays(case["rays"], seed)
    return cam, inc


def _batch_sizes(case):
    """Triangles, image side and photons of each scene of a batch: log-uniform, fixed by the case."""
    rng = np.random.default_rng(case["scenes"] * 1_000_003 + case["tri_hi"])
    out = []
    for _ in range(case["scenes"]):
        tris = math.exp(rng.uniform(math.log(1000), math.log(case["tri_hi"])))
        side = int(round(math.exp(rng.uniform(math.log(64), math.log(case["side_hi"])))))
        out.append((tris, side, 1 << int(rng.integers(14, case["log2_photons_hi"] + 1))))
    return out


def _batch_items(case, seed):
    items = []
    for i, (tris, side, photons) in enumerate(_batch_sizes(case)):
        level = max(0, min(5, int(math.log(tris / 160, 4))))
        cells = max(2, int(math.sqrt(max(tris - 80 * 4 ** level, 8) / 2)))
        items.append((scenes.procedural_scene(width=side, height=side, hf_cells=cells, sphere_level=level,
                                              glass_level=level, seed=seed + 31 * i), photons))
    return items


def prepare(case, seed):
    kind = case["kind"]
    if kind == "trace":
        scene = _scene(case, seed)
        opts = dict(split_alpha=scenes.SOUP_SPLIT_ALPHA, trav_cost=scenes.SOUP_TRAV_COST) if case["split"] else {}
        bvh = api.build_bvh(scene.verts, scene.tri_mat, **opts)
        st = dict(case=case, bvh=bvh)
        for key, r in zip(("cam", "inc"), _rays(case, scene, seed)):
            if r is None:
                continue
            st[key] = torch.from_numpy(r).cuda()
            st[key + "_hit"] = torch.empty(len(r), dtype=torch.int32, device="cuda")
            st[key + "_t"] = torch.empty(len(r), dtype=torch.float32, device="cuda")
        return st
    if kind == "rebuild":
        scene = scenes.soup_scene(case["tris"], seed)
        return dict(case=case, verts=scene.verts, mats=scene.tri_mat,
                    rays=_camera_rays(scene, case["width"], case["height"]))
    if kind == "batch":
        items = _batch_items(case, seed)
        prm = [api.sppm_params(n, alpha=0.7, r0=_r0(s, s.camera.width), seed=seed + i)
               for i, (s, n) in enumerate(items)]
        images = [torch.empty((s.camera.height, s.camera.width), dtype=torch.float32, device="cuda")
                  for s, _ in items]
        return dict(case=case, batch=api.Batch([s for s, _ in items], prm), images=images)
    scene = _scene(case, seed)
    bvh = api.build_bvh(scene.verts, scene.tri_mat)
    if kind == "sppm":
        s = api.sppm_create(scene, _params(case, scene, seed, gather_mode=case["gather"]), bvh=bvh)
        image = torch.empty((case["height"], case["width"]), dtype=torch.float32, device="cuda")
        return dict(case=case, sppm=s, image=image)
    if kind == "render":
        return dict(case=case, scene=scene, params=_params(case, scene, seed), bvh=bvh)
    # diff: the target is an image of the same scene at other albedos, as an inverse-rendering program has it
    rng = np.random.default_rng(seed)
    params = _params(case, scene, seed, record_iterations=case["iters"])
    rho = scene.mat_rho.copy()
    ids = scene.albedo_params
    rho[ids] = np.clip(rho[ids] + rng.uniform(-0.1, 0.1, len(ids)), 0.05, 0.95)
    target = api.render(scene.with_rho(rho), _params(case, scene, seed), case["iters"], bvh=bvh)
    return dict(case=case, scene=scene, params=params, bvh=bvh, target=target, ids=ids,
                albedos=torch.tensor(scene.mat_rho[ids], device="cuda", requires_grad=True),
                Le=torch.tensor(10.0, device="cuda", requires_grad=True))


# ---------------------------------------------------------------------------
# One pass
# ---------------------------------------------------------------------------
def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "trace":
        bvh = state["bvh"]
        if case["call"] == "pair":
            (hi, ti), (hc, tc) = api.trace_rays_multi(bvh, [
                dict(rays=state["inc"], hit=state["inc_hit"], t=state["inc_t"], **INCOHERENT),
                dict(rays=state["cam"], hit=state["cam_hit"], t=state["cam_t"], tile_width=case["width"], **CAMERA)])
            return {"inc_hit": hi, "inc_t": ti, "cam_hit": hc, "cam_t": tc}
        key = "cam" if "cam" in state else "inc"
        rays, hit, t = state[key], state[key + "_hit"], state[key + "_t"]
        if case["call"] == "bucketed":
            api.trace_rays(bvh, rays, hit, t, **INCOHERENT)
        elif case["call"] == "noalloc":
            api.trace_rays_noalloc(bvh, rays, hit, t, **INCOHERENT)
        else:
            api.trace_rays(bvh, rays, hit, t)
        return {"hit": hit, "t": t}
    if kind == "rebuild":
        bvh = api.build_bvh(state["verts"], state["mats"], builder=api.BUILD_GPU_LBVH)
        hit, t = api.trace_rays(bvh, state["rays"])
        bvh.destroy()
        return {"hit": hit, "t": t}
    if kind == "sppm":
        state["sppm"].iterate(case["iters"])
        return {"image": state["sppm"].resolve(state["image"])}
    if kind == "render":
        return {"image": api.render(state["scene"], state["params"], case["iters"], bvh=state["bvh"])}
    if kind == "batch":
        state["batch"].iterate(case["iters"])
        return {"images": state["batch"].resolve(state["images"])}
    albedos, Le = state["albedos"], state["Le"]
    albedos.grad = Le.grad = None
    image = api.sppm_render_diff(albedos, Le, state["scene"], state["ids"], state["params"], case["iters"],
                                 bvh=state["bvh"])
    loss = ((image - state["target"]) ** 2).mean()
    loss.backward()
    return {"image": image.detach(), "loss": loss.detach(), "grad_albedos": albedos.grad, "grad_Le": Le.grad}


# ---------------------------------------------------------------------------
# What a pass cannot do without
# ---------------------------------------------------------------------------
def _n_tri(case):
    if case.get("scene") == "box":
        return 36
    if case.get("scene") == "procedural":
        c, s, g = case.get("cells", 231), case.get("sphere", 5), case.get("glass", 6)
        return 12 + 2 * c * c + 60 * 4 ** s + 20 * 4 ** g
    return case["tris"]


def _ray_flops(n_tri):
    """One ray in a perfect binary hierarchy: a slab test (about 20 operations) per level and one triangle test."""
    return 20 * max(1.0, math.log2(n_tri)) + 60


def work(case):
    kind = case["kind"]
    if kind == "trace":
        n = case["width"] * case["height"] + case["rays"]
        t = _n_tri(case)
        return {"bytes": 40 * n + 36 * t, "flops": n * _ray_flops(t)}
    if kind == "rebuild":
        # vertices once from the host, then one sort of the keys (a comparison per level) and the primary rays
        n, t = case["width"] * case["height"], case["tris"]
        return {"bytes": 40 * n + 40 * t, "flops": n * _ray_flops(t) + t * 20 * math.log2(t)}
    if kind == "batch":
        k = case["iters"]
        sizes = _batch_sizes(case)
        return {"bytes": sum(36 * t + 68 * side * side for t, side, _ in sizes),
                "flops": sum(k * (side * side + 2 * n) * _ray_flops(t) for t, side, n in sizes)}
    t, px, k = _n_tri(case), case["width"] * case["height"], case["iters"]
    # triangles, the per-pixel state read and written once, the image; one eye ray per pixel and two rays per photon
    # path in each iteration; a gradient traces every path a second time
    passes = 2 if kind == "diff" else 1
    return {"bytes": 36 * t + 68 * px + (4 * px if kind == "diff" else 0),
            "flops": passes * k * (px + 2 * case["photons"]) * _ray_flops(t)}


# ---------------------------------------------------------------------------
# 64-bit reference
# ---------------------------------------------------------------------------
def _brute_force_t(verts, rays):
    """Distance of each ray's closest triangle in float64 (+inf: none), Cramer's rule over all pairs."""
    v = torch.from_numpy(verts.astype(np.float64)).cuda()
    r = torch.from_numpy(rays.astype(np.float64)).cuda()
    v0, e1, e2 = v[:, 0], v[:, 1] - v[:, 0], v[:, 2] - v[:, 0]
    nrm = torch.linalg.cross(e1, e2)
    out = torch.empty(len(r), dtype=torch.float64, device="cuda")
    step = max(1, (1 << 22) // len(v))
    for a in range(0, len(r), step):
        o, d = r[a:a + step, None, 0:3], r[a:a + step, None, 4:7]
        det = -(d * nrm).sum(-1)
        s = o - v0
        m = torch.linalg.cross(s, d.expand_as(s))
        t = (s * nrm).sum(-1) / det
        u, w = (e2 * m).sum(-1) / det, -(e1 * m).sum(-1) / det
        ok = (u >= 0) & (w >= 0) & (u + w <= 1) & (t > r[a:a + step, None, 3]) & (t < r[a:a + step, None, 7])
        out[a:a + step] = torch.where(ok, t, torch.inf).amin(1)
    return out


def exact(case, seed):
    if case["kind"] != "trace":
        return None
    n = case["width"] * case["height"] + case["rays"]
    if n * case["tris"] > 1 << 32:
        return None
    scene = _scene(case, seed)
    cam, inc = _rays(case, scene, seed)
    if case["call"] == "pair":
        return {"inc_hit": None, "inc_t": _brute_force_t(scene.verts, inc), "cam_hit": None,
                "cam_t": _brute_force_t(scene.verts, cam)}
    return {"hit": None, "t": _brute_force_t(scene.verts, inc if cam is None else cam)}

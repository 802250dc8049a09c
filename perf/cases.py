"""The framework's work as its users have it: point frames into a voxel map,
the map into planes and polygons, cluster sets into planes and polygons, and
maps into voxel lists.  Sizes are those of the repository's own scenes (the
1.28 m stair cube, the 4x4x2 m local map at 0.01 m, the 0.005 m stress map,
2000 uneven clusters, eight served robots) or lie between them.

A case is a dict; "kind" names the call, the other entries its sizes and
options:

  frame     segment_frame: one frame into the map, the whole map segmented
            (extent, voxel, points, warm frames already in the map, hypotheses,
            fresh: the map is emptied first, labels: per-voxel labels asked
            for, step: the steppable classification, rays: a ray-cast frame
            whose free space is cleared)
  voxelise  clear, insert, export (into the caller's buffers): a cloud
            reduced to its voxels
  clusters  planes and polygons of a caller's cluster set (form: the persistent
            launch or the two-pass calls)
  served    one frame from each of several robots: inserted and labelled map
            by map, planes and polygons of all in one merged pass
  scroll    a robot-centric map: re-centred on the robot, a frame, segmented
"""
import ctypes
import math
import random

import numpy as np
import torch

import paper_2510_01592_amd as vm

EPS = 0.01
MIN_CLUSTER = 30
SEED = 0x5EED
EXTENTS = {"cube": ((0.0, 0.0, -0.64), (1.28, 1.28, 1.28)),      # the stair cube
           "room": ((-2.0, -2.0, -0.1), (4.0, 4.0, 2.0)),        # the local map
           "local": ((-1.2, -1.2, -0.8), (2.4, 2.4, 1.6))}       # the robot-centric grid


def listed():
    return [
        # a small scan on its own: latency and launches are what counts
        {"name": "frame_small_scan", "kind": "frame", "extent": "cube", "voxel": 0.01, "points": 50_000, "warm": 0,
         "hyp": 256, "fresh": True, "labels": True, "step": False, "rays": False},
        # the flagship: a 1M-point frame into a warmed local map
        {"name": "frame_local_map", "kind": "frame", "extent": "room", "voxel": 0.01, "points": 1_000_000, "warm": 8,
         "hyp": 512, "fresh": False, "labels": False, "step": False, "rays": False},
        # a thin frame into a map that has run for a while: thousands of small clusters of accumulated outliers
        {"name": "frame_grown_map", "kind": "frame", "extent": "room", "voxel": 0.01, "points": 230_011, "warm": 40,
         "hyp": 512, "fresh": False, "labels": True, "step": False, "rays": False},
        # the stress map: 0.005 m, 8M points, more hypotheses
        {"name": "frame_fine_map", "kind": "frame", "extent": "room", "voxel": 0.005, "points": 8_000_000, "warm": 2,
         "hyp": 1024, "fresh": False, "labels": False, "step": False, "rays": False},
        # the paper's whole path: steppable classification, gated clustering, planes, polygons
        {"name": "frame_steppable", "kind": "frame", "extent": "room", "voxel": 0.01, "points": 1_000_000, "warm": 8,
         "hyp": 512, "fresh": False, "labels": True, "step": True, "rays": False},
        # what a sensor sees from where it stands, with free space cleared along its rays
        {"name": "frame_clearing", "kind": "frame", "extent": "room", "voxel": 0.01, "points": 1_000_000, "warm": 4,
         "hyp": 512, "fresh": False, "labels": False, "step": False, "rays": True},
        # a depth-camera cloud reduced to voxels, below the grouped insert's threshold
        {"name": "voxelise_small", "kind": "voxelise", "extent": "cube", "voxel": 0.01, "points": 20_011},
        # an accumulated cloud reduced to voxels
        {"name": "voxelise_large", "kind": "voxelise", "extent": "room", "voxel": 0.01, "points": 4_000_003},
        # thousands of clusters of very uneven size in one launch
        {"name": "clusters_2000", "kind": "clusters", "clusters": 2000, "n_min": 50, "n_max": 200_000, "hyp": 1024,
         "form": "persistent"},
        # a handful of clusters, the paper's hypothesis count
        {"name": "clusters_16", "kind": "clusters", "clusters": 16, "n_min": 10_000, "n_max": 30_000, "hyp": 100,
         "form": "two_pass"},
        # eight robots' frames, planes and polygons in one merged pass
        {"name": "served_8", "kind": "served", "robots": 8, "n_min": 200_000, "n_max": 2_000_000, "warm": 4,
         "hyp": 512},
        # the robot-centric map follows its robot
        {"name": "scroll_local", "kind": "scroll", "points": 300_000, "warm": 4, "hyp": 256},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["frame", "frame", "frame", "voxelise", "clusters", "clusters", "served", "scroll"])
    if kind == "frame":
        ext = rng.choice(["cube", "room", "room"])
        step = rng.random() < 0.2
        rays = not step and rng.random() < 0.25
        fine = ext == "room" and not step and not rays and rng.random() < 0.2
        return {"kind": "frame", "extent": ext, "voxel": 0.005 if fine else rng.choice([0.01, 0.01, 0.012, 0.02]),
                "points": _log_int(rng, 10_000, 200_000) if ext == "cube" else _log_int(rng, 50_000, 2_000_000),
                "warm": rng.randint(0, 3) if ext == "cube" else rng.randint(1, 12),
                "hyp": rng.choice([100, 200, 256, 512, 1024]), "fresh": ext == "cube" and rng.random() < 0.5,
                "labels": rng.random() < 0.5, "step": step, "rays": rays}
    if kind == "voxelise":
        ext = rng.choice(["cube", "room"])
        return {"kind": "voxelise", "extent": ext, "voxel": rng.choice([0.01, 0.015, 0.02]),
                "points": _log_int(rng, 5_000, 4_000_000)}
    if kind == "clusters":
        persistent = rng.random() < 0.6
        lo = _log_int(rng, 40, 4_000)
        hi = min(200_000, _log_int(rng, 4 * lo, 100 * lo))
        return {"kind": "clusters", "clusters": _log_int(rng, 1, 1500 if persistent else 200), "n_min": lo,
                "n_max": hi, "hyp": rng.choice([100, 256, 512, 1000]),
                "form": "persistent" if persistent else "two_pass"}
    if kind == "served":
        return {"kind": "served", "robots": rng.randint(2, 8), "n_min": 200_000,
                "n_max": rng.randint(300_000, 2_000_000), "warm": rng.randint(2, 4), "hyp": rng.choice([256, 512])}
    return {"kind": "scroll", "points": _log_int(rng, 100_000, 500_000), "warm": rng.randint(2, 6),
            "hyp": rng.choice([100, 256])}


# ---- inputs ---------------------------------------------------------------------
def _tilt(rng, deg):
    a, b = (math.radians(rng.uniform(-deg, deg)) for _ in range(2))
    ca, sa, cb, sb = math.cos(a), math.sin(a), math.cos(b), math.sin(b)
    return np.array([[cb, 0.0, sb], [sa * sb, ca, -sa * cb], [-ca * sb, sa, ca * cb]])


def _hrect(x0, x1, y0, y1, z):
    return ((x0 + x1) / 2, (y0 + y1) / 2, z), (1, 0, 0), (0, 1, 0), (x1 - x0) / 2, (y1 - y0) / 2


def _scene(extent, fine, rng):
    """Rectangles (centre, axis, axis, half, half) as float64 device tensors:
    floor, steps, tables, and tilted patches (yawed boxes on the fine map)
    kept apart from everything else by their bounding boxes."""
    if extent == "cube":
        rs = [_hrect(0.0, 1.28, 0.0, 1.28, 0.0), _hrect(0.40, 0.70, 0.34, 0.94, 0.18),
              _hrect(0.70, 1.00, 0.34, 0.94, 0.36)]
    else:
        rs = [_hrect(-2.0, 2.0, -2.0, 2.0, 0.0)]
        rs += [_hrect(-1.5 + 0.28 * i, -1.22 + 0.28 * i, -1.9, -0.9, 0.18 * (i + 1)) for i in range(12)]
        rs += [_hrect(0.3, 1.5, 0.5, 1.3, 0.72)]
        boxes = []
        for c, a, b, ha, hb in rs:
            r = np.abs(np.array(a)) * ha + np.abs(np.array(b)) * hb
            boxes.append((np.array(c) - r, np.array(c) + r))
        want, tries = (400 if fine else 20), 0
        placed = 0
        while placed < want and tries < 6000:
            tries += 1
            c = np.array([rng.uniform(-1.8, 1.8), rng.uniform(-1.8, 1.8), rng.uniform(0.1, 1.6)])
            if fine:
                h = np.array([rng.uniform(0.025, 0.2) for _ in range(3)])
                yaw = rng.uniform(0, 2 * math.pi)
                ax = np.array([[math.cos(yaw), math.sin(yaw), 0], [-math.sin(yaw), math.cos(yaw), 0], [0, 0, 1]])
                new = [(c + s * h[i] * ax[i], ax[(i + 1) % 3], ax[(i + 2) % 3], h[(i + 1) % 3], h[(i + 2) % 3])
                       for i in range(3) for s in (1.0, -1.0)]
                r = np.abs(ax * h[:, None]).sum(0)
            else:
                t = _tilt(rng, 30)
                ha, hb = rng.uniform(0.1, 0.3), rng.uniform(0.1, 0.3)
                new = [(c, t[:, 0], t[:, 1], ha, hb)]
                r = np.abs(t[:, 0]) * ha + np.abs(t[:, 1]) * hb
            lo, hi = c - r - 0.04, c + r + 0.04
            if lo[2] < 0.0 or hi[2] > 1.9 or any((lo < b[1]).all() and (hi > b[0]).all() for b in boxes):
                continue
            boxes.append((c - r, c + r))
            rs += new
            placed += 1
    cols = [np.array([r[i] for r in rs], np.float64) for i in range(5)]
    return [torch.from_numpy(x).cuda() for x in cols]


def _gen(seed, n):
    g = torch.Generator(device="cuda")
    g.manual_seed((int(seed) * 1_000_003 + n) & 0x7FFFFFFF)
    return g


def _rand(g, *shape):
    return torch.rand(*shape, dtype=torch.float64, device="cuda", generator=g)


def _randn(g, *shape):
    return torch.randn(*shape, dtype=torch.float64, device="cuda", generator=g)


def _surface_frame(scene, extent, n, sigma, g, outliers=0.05):
    """n points (map frame, float64): uniform over the surfaces with noise along
    the normals, and a fraction anywhere in the extent."""
    C, A, B, ha, hb = scene
    lo, size = (torch.tensor(v, dtype=torch.float64, device="cuda") for v in EXTENTS[extent])
    w = torch.multinomial((ha * hb).float(), n, replacement=True, generator=g)
    s = 2.0 * _rand(g, n, 2) - 1.0
    p = C[w] + (s[:, :1] * ha[w, None]) * A[w] + (s[:, 1:] * hb[w, None]) * B[w]
    p += sigma * _randn(g, n, 1) * torch.linalg.cross(A, B)[w]
    out = _rand(g, n) < outliers
    return torch.where(out[:, None], lo + size * _rand(g, n, 3), p)


def _ray_frame(scene, sensor, n, sigma, g, outliers=0.05):
    """n returns of rays from the sensor (map frame): the first surface hit,
    some of them spurious and early."""
    C, A, B, ha, hb = scene
    N = torch.linalg.cross(A, B)
    o = torch.tensor(sensor, dtype=torch.float64, device="cuda")
    d = _randn(g, 2 * n + 4096, 3)
    d /= d.norm(dim=1, keepdim=True)
    best = torch.full((len(d),), math.inf, dtype=torch.float64, device="cuda")
    for j in range(len(ha)):
        t = ((C[j] - o) @ N[j]) / (d @ N[j])
        q = o + t[:, None] * d - C[j]
        ok = (t > 1e-6) & (t < best) & (t <= 8.0) & ((q @ A[j]).abs() <= ha[j]) & ((q @ B[j]).abs() <= hb[j])
        best = torch.where(ok, t, best)
    # the hits come round again if the scene returned fewer than n
    hit = torch.nonzero(torch.isfinite(best)).flatten()
    hit = hit[torch.arange(n, device="cuda") % len(hit)]
    t = best[hit]
    r = t + sigma * _randn(g, n)
    r = torch.where(_rand(g, n) < outliers, t * (0.05 + 0.9 * _rand(g, n)), r)
    return o + r[:, None] * d[hit]


def _pose(rng, step_t=0.02, step_deg=0.5):
    """A sensor's pose: a small rotation and translation."""
    w = [math.radians(rng.gauss(0, step_deg)) for _ in range(3)]
    cx, sx, cy, sy, cz, sz = (f(v) for v in w for f in (math.cos, math.sin))
    R = (np.array([[cz, -sz, 0], [sz, cz, 0], [0, 0, 1.0]]) @ np.array([[cy, 0, sy], [0, 1.0, 0], [-sy, 0, cy]])
         @ np.array([[1.0, 0, 0], [0, cx, -sx], [0, sx, cx]]))
    return R, np.array([rng.gauss(0, step_t) for _ in range(3)])


def _to_sensor(p, R, t):
    R, t = torch.from_numpy(np.ascontiguousarray(R)).cuda(), torch.from_numpy(t).cuda()
    return ((p - t) @ R).float().contiguous()


def _dims(extent, voxel):
    return tuple(max(1, int(round(s / voxel))) for s in EXTENTS[extent][1])


def _hash_log2(case):
    if case["kind"] == "scroll":
        return 21
    if case["kind"] == "voxelise" or case.get("extent") == "cube":
        n = case["points"] * (1 + case.get("warm", 0))
    else:
        n = min(case["points"] * (1 + case.get("warm", 0)), 3_500_000 if case["voxel"] >= 0.01 else 16_000_000)
    return max(16, min(25, math.ceil(math.log2(2 * n))))


def _outputs(k_cap, n_cap, hyp):
    return vm.PlaneBuffers.alloc(k_cap, n_cap, hyp), vm.HullBuffers.alloc(k_cap, max(1, n_cap // 2))


def prepare(case, seed):
    rng = random.Random(seed)
    kind = case["kind"]
    if kind == "clusters":
        off, xyz, tag = _cluster_points(case, seed)
        K, N = case["clusters"], int(off[-1])
        own = {"off": off.to(torch.int32), "tag": tag, "meta": torch.tensor([K, N], dtype=torch.int32, device="cuda")}
        for i, a in enumerate("xyz"):
            own[a] = xyz[:, i].contiguous()
        view = vm.cluster_view(own["off"], own["x"], own["y"], own["z"], own["tag"], own["meta"])
        planes, hulls = _outputs(K, N, case["hyp"])
        work = torch.empty(vm.workspace_bytes(K, N, case["hyp"]), dtype=torch.uint8, device="cuda")
        return {"case": case, "view": view, "own": own, "planes": planes, "hulls": hulls, "work": work}
    if kind == "served":
        n = case["robots"]
        st = {"case": case, "maps": [], "frames": [], "poses": [], "planes": [], "hulls": []}
        for r in range(n):
            one = {"kind": "frame", "extent": "room", "voxel": 0.01, "points": rng.randint(case["n_min"], case["n_max"]),
                   "warm": case["warm"], "hyp": case["hyp"], "fresh": False, "labels": False, "step": False,
                   "rays": False}
            m, xyz, R, t = _map_and_frame(one, seed * 16 + r, rng, 23)
            st["maps"].append(m)
            st["frames"].append(xyz)
            st["poses"].append((R, t))
            planes, hulls = _outputs(8192, 1 << 21, case["hyp"])
            st["planes"].append(planes)
            st["hulls"].append(hulls)
        st["k_cap"], st["n_cap"] = 32768, 1 << 23
        st["work"] = torch.empty(vm.multi_workspace_bytes(st["k_cap"], st["n_cap"], case["hyp"]), dtype=torch.uint8,
                                 device="cuda")
        return st
    if kind == "scroll":
        # the robot walks to and fro; the map holds what it saw at both ends
        scene = _scene("room", False, rng)
        ends = [(0.30, -0.20, 0.60), (0.55, 0.05, 0.62)]
        m = vm.Map(EXTENTS["local"][0], 0.01, _dims("local", 0.01), _hash_log2(case))
        g = _gen(seed, 1)
        frames = []
        for i in range(case["warm"] + 2):
            p = _surface_frame(scene, "room", case["points"], 0.003, g).float().contiguous()
            m.recenter(ends[i % 2])
            if i < case["warm"]:
                m.insert(p)
            else:
                frames.append(p)
        planes, hulls = _outputs(4096, 1 << 20, case["hyp"])
        return {"case": case, "map": m, "frames": frames, "ends": ends, "turn": 0, "planes": planes, "hulls": hulls}
    m, xyz, R, t = _map_and_frame(case, seed, rng, _hash_log2(case))
    st = {"case": case, "map": m, "xyz": xyz, "R": R, "t": t}
    if kind == "voxelise":
        # the list's buffers, as many rows as the cloud has points
        n = case["points"]
        st["key"] = torch.zeros(n, dtype=torch.int32, device="cuda")
        st["count"] = torch.zeros(n, dtype=torch.int32, device="cuda")
        st["sums"] = torch.zeros((n, 3), dtype=torch.int64, device="cuda")
        st["mean"] = torch.zeros((n, 3), dtype=torch.float32, device="cuda")
        st["n"] = ctypes.c_uint64()
    if kind == "frame":
        cap = 1 << _hash_log2(case)
        st["planes"], st["hulls"] = _outputs(min(65536, cap // MIN_CLUSTER + 1), cap // 2, case["hyp"])
        st["labels"] = torch.zeros(cap, dtype=torch.int32, device="cuda") if case["labels"] else None
        st["step"] = vm.step_params() if case["step"] else None
    return st


def _frames_of(case, seed, rng):
    """The warm frames' and the case's own points in the map frame, and its sensor pose."""
    fine = case["voxel"] < 0.01
    scene = _scene(case["extent"], fine, rng)
    sigma = 0.0015 if fine else 0.002 if case["extent"] == "cube" else 0.003
    out = 0.02 if case["extent"] == "cube" else 0.05
    n, warm = case["points"], case.get("warm", 0)
    R, t = _pose(rng) if case["kind"] == "frame" else (np.eye(3), np.zeros(3))
    if case.get("rays"):
        t = t + ((0.2, -0.3, 1.0) if case["extent"] == "room" else (0.3, 0.3, 0.5))
    for i in range(warm + 1):
        g = _gen(seed, i)
        # a map is warmed by whole frames, whatever the size of the one that follows
        k = n if i == warm or case["extent"] == "cube" else max(n, 1_000_000)
        if case.get("rays"):
            yield _ray_frame(scene, t, k, sigma, g, out), R, t
        else:
            yield _surface_frame(scene, case["extent"], k, sigma, g, out), R, t


def _map_and_frame(case, seed, rng, log2):
    m = vm.Map(EXTENTS[case["extent"]][0], case["voxel"], _dims(case["extent"], case["voxel"]), log2)
    last = None
    for p, R, t in _frames_of(case, seed, rng):
        if last is not None:
            m.insert(last, R, t)
        last = _to_sensor(p, R, t)
    return m, last, R, t


def _cluster_points(case, seed):
    """Noisy plane patches of log-uniform size, a tenth of each off its plane."""
    K = case["clusters"]
    # the sizes belong to the case: buffers are sized by them
    n = torch.exp(math.log(case["n_min"]) + (math.log(case["n_max"]) - math.log(case["n_min"])) * _rand(_gen(3, K), K))
    n = n.long()
    g = _gen(seed, 7)
    off = torch.zeros(K + 1, dtype=torch.int64, device="cuda")
    off[1:] = torch.cumsum(n, 0)
    N = int(off[-1])
    ct = math.cos(math.radians(40)) + (1 - math.cos(math.radians(40))) * _rand(g, K)
    ph = 2 * math.pi * _rand(g, K)
    st = torch.sqrt(1 - ct * ct)
    nrm = torch.stack([st * torch.cos(ph), st * torch.sin(ph), ct], 1)
    a = torch.linalg.cross(nrm, torch.tensor([1.0, 0, 0], dtype=torch.float64, device="cuda").expand_as(nrm))
    a /= a.norm(dim=1, keepdim=True)
    b = torch.linalg.cross(nrm, a)
    c = torch.tensor([-2.0, -2.0, 0.0], dtype=torch.float64, device="cuda") + _rand(g, K, 3) * torch.tensor(
        [4.0, 4.0, 2.0], dtype=torch.float64, device="cuda")
    xyz = torch.empty(N, 3, dtype=torch.float32, device="cuda")
    owner = torch.repeat_interleave(torch.arange(K, device="cuda"), n)
    for i in range(0, N, 1 << 23):   # in slices: the temporaries stay small
        w = owner[i:i + (1 << 23)]
        m = len(w)
        half = 0.005 * torch.sqrt(n[w].double())
        s = 2.0 * _rand(g, m, 2) - 1.0
        far = _rand(g, m) < 0.1
        h = torch.where(far, 0.2 * _rand(g, m) - 0.1, 0.002 * _randn(g, m))
        xyz[i:i + m] = (c[w] + (s[:, 0] * half)[:, None] * a[w] + (s[:, 1] * half)[:, None] * b[w]
                        + h[:, None] * nrm[w]).float()
    return off, xyz, torch.arange(K, dtype=torch.int32, device="cuda") * 7919 + 3


# ---- one pass ---------------------------------------------------------------------
def _result(planes, hulls):
    return {"plane": planes.plane, "best": planes.best_h, "inliers": planes.n_inliers, "in_off": planes.in_off,
            "in_idx": planes.in_idx, "status": planes.status, "v_off": hulls.v_off, "v_idx": hulls.v_idx,
            "v_xyz": hulls.v_xyz, "area": hulls.area, "hstatus": hulls.status}


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "frame":
        if case["fresh"]:
            state["map"].clear()
        state["map"].segment_frame(state["xyz"], state["planes"], state["hulls"], R=state["R"], t=state["t"],
                                   min_cluster=MIN_CLUSTER, n_hyp=case["hyp"], eps=EPS, seed=SEED, frame=0,
                                   labels=state["labels"], step=state["step"], clear=case["rays"])
        r = _result(state["planes"], state["hulls"])
        if state["labels"] is not None:
            r["labels"] = state["labels"]
        return r
    if kind == "voxelise":
        state["map"].clear()
        state["map"].insert(state["xyz"])
        out = {k: state[k] for k in ("key", "count", "sums", "mean")}
        st = vm.lib().vm_map_export(state["map"].handle, *(t.data_ptr() for t in out.values()), case["points"],
                                    ctypes.byref(state["n"]), torch.cuda.current_stream().cuda_stream)
        if st != vm.VM_OK:
            raise vm.VMError(st, "vm_map_export")
        return dict(out, voxels=int(state["n"].value))
    if kind == "clusters":
        p = vm.ransac_params(case["hyp"], EPS, SEED, 0)
        if case["form"] == "persistent":
            vm.planes_hulls(state["view"], p, state["planes"], state["hulls"], state["work"])
        else:
            vm.ransac_planes(state["view"], p, state["planes"], state["work"])
            vm.hulls(state["view"], state["planes"], state["hulls"], state["work"])
        return _result(state["planes"], state["hulls"])
    if kind == "served":
        views = []
        for m, xyz, (R, t) in zip(state["maps"], state["frames"], state["poses"]):
            m.insert(xyz, R, t)
            views.append(m.ccl(MIN_CLUSTER))
        vm.planes_hulls_multi(views, list(range(len(views))), vm.ransac_params(case["hyp"], EPS, SEED, 0),
                              state["planes"], state["hulls"], state["k_cap"], state["n_cap"], state["work"])
        return [{k: r[k] for k in ("plane", "best", "in_off", "in_idx", "v_off", "v_xyz", "area")}
                for r in (_result(p, h) for p, h in zip(state["planes"], state["hulls"]))]
    i = state["turn"]
    state["turn"] = 1 - i
    state["map"].recenter(state["ends"][i])
    state["map"].segment_frame(state["frames"][i], state["planes"], state["hulls"], min_cluster=MIN_CLUSTER,
                               n_hyp=case["hyp"], eps=EPS, seed=SEED, frame=0)
    return _result(state["planes"], state["hulls"])


# ---- what a pass cannot do without ------------------------------------------------
def _frame_work(voxels, points, hyp, labels=False, step=False, rays=False):
    """Points in; a slot of 32 bytes read and written for the voxels a frame
    touches; parents, keys and means of all voxels written and read once; three
    fused multiply-adds per (clustered voxel, hypothesis)."""
    kept = 0.45 * voxels
    b = 12 * points + 64 * min(points, kept) + 20 * voxels + 20 * kept + (4 * voxels if labels else 0)
    f = 6.0 * kept * hyp
    if step:
        b += 33 * voxels
        f += 4000.0 * voxels
    if rays:
        b += 12 * points
        f += 10.0 * 200 * points
    return b, f


def _voxels(case):
    cube = case["extent"] == "cube"
    surface = (2.0 if cube else 26.0) / case["voxel"] ** 2 * 2.0 * (2.5 if case["voxel"] < 0.01 else 1.0)
    frames = 1 + case.get("warm", 0)
    per = max(case["points"], 1_000_000) if not cube else case["points"]
    return min(surface, frames * per) + (0.02 if cube else 0.0 if case.get("rays") else 0.05) * frames * per


def work(case):
    kind = case["kind"]
    if kind == "frame":
        b, f = _frame_work(_voxels(case), case["points"], case["hyp"], case["labels"], case["step"], case["rays"])
    elif kind == "voxelise":
        v = min(_voxels(dict(case, warm=0)), case["points"])
        b, f = 12 * case["points"] + 64 * v + 44 * v, 30.0 * case["points"]
    elif kind == "clusters":
        n = case["clusters"] * (case["n_max"] - case["n_min"]) / max(1e-9, math.log(case["n_max"] / case["n_min"]))
        b, f = 12 * n + 4 * n, 6.0 * n * case["hyp"]
    elif kind == "served":
        n = (case["n_min"] + case["n_max"]) / 2
        one = _frame_work(600_000 + 50_000 * case["warm"], n, case["hyp"])
        b, f = case["robots"] * one[0], case["robots"] * one[1]
    else:
        b, f = _frame_work(400_000, case["points"], case["hyp"])
        b += 64 * 400_000
    return {"bytes": float(b), "flops": float(f)}


# ---- the same in 64 bits -------------------------------------------------------------
def exact(case, seed):
    """The floating outputs from the definitions: voxel means; planes, polygon
    vertices and areas of cluster sets and of the frames on the small grid.
    (Which hypothesis wins is a matter of whole numbers: the inlier counts of
    the stated 32-bit test.)  None where that would take long."""
    kind = case["kind"]
    if kind == "voxelise":
        rng = random.Random(seed)
        (p, R, t), = _frames_of(case, seed, rng)
        x = _to_sensor(p, R, t).double().cpu().numpy()
        cell = _voxel_sums(case, [x])[2]
        mean = np.zeros((case["points"], 3))
        mean[:len(cell)] = cell
        return {"key": None, "count": None, "sums": None, "mean": mean, "voxels": None}
    if kind == "clusters":
        off, xyz, tag = _cluster_points(case, seed)
        if int(off[-1]) * case["hyp"] > 100_000_000 or int(off[-1]) > 400_000:
            return None
        off, xyz = off.cpu().numpy(), xyz.cpu().numpy()
        K, N = case["clusters"], len(xyz)
        return _floats(_planes(off, xyz, tag.cpu().numpy().view(np.uint32), case["hyp"]), K, max(1, N // 2))
    if kind == "frame" and case["extent"] == "cube" and not case["step"] and not case["rays"] \
            and case["points"] * (1 + case["warm"]) <= 300_000:
        rng = random.Random(seed)
        clouds = []
        for p, R, t in _frames_of(case, seed, rng):
            x = _to_sensor(p, R, t).double().cpu().numpy()
            clouds.append(np.stack([(t[i] + R[i, 0] * x[:, 0]) + R[i, 1] * x[:, 1] + R[i, 2] * x[:, 2]
                                    for i in range(3)], 1))
        key, _, _, mean = _voxel_sums(case, clouds[-1:] if case["fresh"] else clouds)
        lab = _labels(key, _dims(case["extent"], case["voxel"]))
        root, inv, n = np.unique(lab, return_inverse=True, return_counts=True)
        keep = n >= MIN_CLUSTER
        order = np.argsort(inv, kind="stable")
        order = order[keep[inv[order]]]
        off = np.concatenate([[0], np.cumsum(n[keep])])
        r = _floats(_planes(off, mean[order], root[keep].astype(np.uint32), case["hyp"]),
                    min(65536, (1 << _hash_log2(case)) // MIN_CLUSTER + 1), (1 << _hash_log2(case)) // 4)
        if case["labels"]:
            r["labels"] = None
        return r
    return None


def _voxel_sums(case, clouds):
    """Occupied voxels by key: counts, the mean of the points in 64 bits, and
    the stored mean (a whole number of 2^-20 voxels) as float32."""
    o, s, dims = np.array(EXTENTS[case["extent"]][0]), case["voxel"], np.array(_dims(case["extent"], case["voxel"]))
    p = np.concatenate(clouds)
    f = np.floor((p - o) * (1048576.0 / s))
    ok = ((f >= 0) & (f < dims * 1048576.0)).all(1)
    q, p = f[ok].astype(np.int64), p[ok]
    v = q >> 20
    k = v[:, 0] + dims[0] * (v[:, 1] + dims[1] * v[:, 2])
    key, inv, cnt = np.unique(k, return_inverse=True, return_counts=True)
    cell = np.stack([np.bincount(inv, weights=p[:, i], minlength=len(key)) / cnt for i in range(3)], 1)
    at = np.stack([key % dims[0], key // dims[0] % dims[1], key // (dims[0] * dims[1])], 1)
    off = np.stack([np.bincount(inv, weights=(q[:, i] & 0xFFFFF).astype(np.float64), minlength=len(key))
                    for i in range(3)], 1).astype(np.int64) // cnt[:, None]
    return key, cnt, cell, ((at + off * 2.0 ** -20) * s + o).astype(np.float32)


def _labels(key, dims):
    """Smallest key of each 26-connected component."""
    x, y, z = key % dims[0], key // dims[0] % dims[1], key // (dims[0] * dims[1])
    edges = []
    for dz in (-1, 0):
        for dy in (-1, 0, 1):
            for dx in (-1, 0, 1):
                if (dz, dy, dx) >= (0, 0, 0):
                    continue
                inside = (x + dx >= 0) & (x + dx < dims[0]) & (y + dy >= 0) & (y + dy < dims[1]) & (z + dz >= 0)
                nb = key + dx + dims[0] * (dy + dims[1] * dz)
                at = np.minimum(np.searchsorted(key, nb), len(key) - 1)
                hit = np.nonzero(inside & (key[at] == nb))[0]
                edges.append((hit, at[hit]))
    a, b = (np.concatenate(e) for e in zip(*edges))
    lab = np.arange(len(key))
    while True:
        new = lab.copy()
        m = np.minimum(lab[a], lab[b])
        np.minimum.at(new, lab[a], m)
        np.minimum.at(new, lab[b], m)
        new = new[new]
        if (new == lab).all():
            return key[lab]
        lab = new


def _philox(h, tag):
    """Three 32-bit draws of hypothesis h of a cluster."""
    g = np.random.Philox(counter=0, key=0)
    s = g.state
    at = (h + (tag << 64) - 1) % (1 << 256)   # the generator steps its counter before it draws
    s["state"]["key"] = np.array([SEED, 0], np.uint64)
    s["state"]["counter"] = np.array([(at >> 64 * i) & 0xFFFFFFFFFFFFFFFF for i in range(4)], np.uint64)
    s["buffer_pos"], s["has_uint32"] = 4, 0
    g.state = s
    return [int(v) >> 32 for v in g.random_raw(3)]


def _planes(off, xyz, tag, hyp):
    """Per cluster: the winning plane, its polygon's vertices on the plane, and
    the polygon's area."""
    res = []
    eps = np.float32(EPS)
    for k in range(len(off) - 1):
        P = xyz[off[k]:off[k + 1]]
        n = len(P)
        best, plane, inl = 0, None, None
        D = P.astype(np.float64)
        for h in range(hyp if n >= 3 else 0):
            u = _philox(h, int(tag[k]))
            i = (u[0] * n) >> 32
            j = (u[1] * (n - 1)) >> 32
            j += j >= i
            l = (u[2] * (n - 2)) >> 32
            l += l >= min(i, j)
            l += l >= max(i, j)
            nr = np.cross(D[j] - D[i], D[l] - D[i])
            if nr @ nr < 1e-24:
                continue
            nr = nr / np.sqrt(nr @ nr)
            if tuple(nr[::-1]) < (0.0, 0.0, 0.0):
                nr = -nr
            pl = np.append(nr, -(nr @ D[i]))
            w = pl.astype(np.float32).astype(np.float64)
            d = (w[0] * D[:, 0] + w[3]).astype(np.float32).astype(np.float64)
            d = (w[1] * D[:, 1] + d).astype(np.float32).astype(np.float64)
            d = (w[2] * D[:, 2] + d).astype(np.float32)
            hit = np.abs(d) < eps
            c = int(hit.sum())
            if plane is None or c > best:
                best, plane, inl = c, pl, np.nonzero(hit)[0]
        res.append((plane, *_polygon(plane, D, inl)) if plane is not None else (np.zeros(4), np.zeros((0, 3)), 0.0))
    return res


def _polygon(plane, D, inl):
    if not len(inl):
        return np.zeros((0, 3)), 0.0
    n = plane[:3].astype(np.float32).astype(np.float64)
    d = float(np.float32(plane[3]))
    a = np.array([1.0, 0, 0]) if abs(n[0]) < 0.9 else np.array([0, 1.0, 0])
    u = np.cross(a, n)
    u /= np.sqrt(u @ u)
    v = np.cross(n, u)
    Q = D[inl]
    E = Q - Q[0]
    U, V = E @ u, E @ v
    order = np.lexsort((np.arange(len(U)), V, U))

    def chain(idx):
        s = []
        for i in idx:
            while len(s) >= 2 and (U[s[-1]] - U[s[-2]]) * (V[i] - V[s[-2]]) - (V[s[-1]] - V[s[-2]]) * (
                    U[i] - U[s[-2]]) <= 0.0:
                s.pop()
            s.append(i)
        return s
    lo, up = chain(order.tolist()), chain(order.tolist()[::-1])
    s = lo + up[1:-1]
    area = 0.5 * sum(U[s[i - 1]] * V[s[i]] - U[s[i]] * V[s[i - 1]] for i in range(len(s))) if len(s) >= 3 else 0.0
    X = Q[s]
    return X - (X @ n + d)[:, None] * n, area


def _floats(res, k_cap, v_cap):
    plane, area, xyz = np.zeros((k_cap, 4)), np.zeros(k_cap), np.zeros((v_cap, 3))
    at = 0
    for k, (p, v, a) in enumerate(res):
        plane[k], area[k] = p, a
        xyz[at:at + len(v)] = v
        at += len(v)
    return {"plane": plane, "best": None, "inliers": None, "in_off": None, "in_idx": None, "status": None,
            "v_off": None, "v_idx": None, "v_xyz": xyz, "area": area, "hstatus": None}

"""Cases that stand for what programs do with this library on one GPU.

A LiDAR mapping program ingests scans (voxel maps), decides by overlap which
frames to connect, binds the factors of a local submap or of the global graph
to their clouds and maps, and then linearizes them round after round inside an
optimizer, directly or through the batching server.  The cases follow the
workloads of bench.py (one 2,000-point factor, 500 and 4,500 scan factors, the
local-mapping and serving streams) in sizes and options, on scans ray-cast on
the GPU: 64 rings x 1,024 azimuths in a street of facades and poles, range
noise 2 cm, plane-like covariances (1, 1, 1e-3) about noisy normals, poses off
the truth by 0.1 m / 2 degrees (global) or 2 cm / 0.2 degrees (local).
"""

import math
import random

import numpy as np
import torch

from paper_2109_07073_amd import vgicp as vg


def listed():
    return [
        # One small factor, replayed as a graph: the latency of a single relinearization.
        {"name": "single_factor", "kind": "round", "scene": "room", "frames": 2, "factors": 1,
         "lo": 2000, "hi": 2000, "target": 2000, "resolution": 1.0, "tile": 0, "layout": "grouped",
         "reorder": False, "graph": True, "accum": "mixed", "form": "auto"},
        # Factors of a mapping batch (sources of 5,000 to 40,000 points) with every sum in FP64.
        {"name": "round48_f64", "kind": "round", "scene": "street", "frames": 40, "factors": 48,
         "lo": 5000, "hi": 40000, "target": 20000, "resolution": 0.5, "tile": 0,
         "layout": "grouped", "reorder": False, "graph": False, "accum": "f64", "form": "auto"},
        # A pose graph of 100 scans as the factor set is created, no tuning: each frame is the
        # source of about five factors.
        {"name": "round500", "kind": "round", "scene": "street", "frames": 100, "factors": 500,
         "lo": 0, "hi": 0, "target": 20000, "resolution": 0.5, "tile": 0, "layout": "grouped",
         "reorder": False, "graph": True, "accum": "mixed", "form": "auto"},
        # The global graph: 4,500 factors with their own sources, target-order copies and the
        # balanced tile table, replayed as a graph.
        {"name": "round4500", "kind": "round", "scene": "street", "frames": 1000,
         "factors": 4500, "lo": 5000, "hi": 40000, "target": 20000, "resolution": 0.5,
         "tile": 13824, "layout": "balanced", "reorder": True, "graph": True, "accum": "mixed",
         "form": "auto"},
        # The trial step of an optimizer over the 500-factor graph: costs only.
        {"name": "cost500", "kind": "cost", "frames": 100, "factors": 500, "target": 20000,
         "resolution": 0.5},
        # Overlap of every pair when a graph's factors are created.
        {"name": "overlap500", "kind": "overlap", "frames": 100, "factors": 500, "target": 20000,
         "resolution": 0.5},
        # One iteration of a submap's optimizer: fully connected frames, linearize, assemble
        # the linear system, cost at the trial poses.
        {"name": "submap_iteration", "kind": "iteration", "frames": 10, "target": 20000,
         "resolution": 0.5},
        # A closed submap becomes a factor graph: voxel maps, factor set, first linearization.
        {"name": "submap_build", "kind": "build", "frames": 10, "target": 20000,
         "resolution": 0.5},
        # An arriving keyframe is voxelized (an odd number of returns).
        {"name": "voxelize_scan", "kind": "voxelize", "points": 20011, "resolution": 0.5},
        # A merged submap of 16 scans is voxelized.
        {"name": "voxelize_submap", "kind": "voxelize", "points": 320000, "resolution": 0.5},
        # A new keyframe is checked against the resident maps.
        {"name": "connect200", "kind": "connect", "frames": 200, "target": 20000,
         "resolution": 0.5},
        # One round of two optimizers on the server: the factors of the newest 20 keyframes and
        # a fully connected graph of the newest 10.
        {"name": "serving_round", "kind": "serving", "frames": 50, "target": 20000, "window": 20,
         "reach": 29, "local": 10, "resolution": 0.5},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng: random.Random):
    kind = rng.choice(["round", "round", "round", "cost", "overlap", "iteration", "build",
                       "voxelize", "voxelize", "connect", "serving"])
    r = rng.choice([0.25, 0.5, 0.5, 1.0])
    if kind == "voxelize":
        return {"kind": kind, "points": _log_int(rng, 500, 320000), "resolution": r}
    pts = _log_int(rng, 2000, 30000)
    if kind in ("iteration", "build"):
        return {"kind": kind, "frames": rng.randint(2, 16), "target": pts, "resolution": r}
    if kind == "connect":
        return {"kind": kind, "frames": _log_int(rng, 2, 400), "target": pts, "resolution": r}
    if kind == "serving":
        return {"kind": kind, "frames": rng.randint(12, 60), "target": pts,
                "window": rng.randint(4, 20), "reach": rng.randint(5, 29),
                "local": rng.randint(2, 12), "resolution": r}
    factors = _log_int(rng, 1, 1500)
    frames = max(3, math.ceil(factors / rng.uniform(4.0, 8.0)))
    if kind in ("cost", "overlap"):
        return {"kind": kind, "frames": frames, "factors": min(factors, frames * (frames - 1) // 2),
                "target": pts, "resolution": r}
    own = rng.random() < 0.5
    accum = rng.choice(["mixed", "mixed", "mixed", "f64", "f32_comp"])
    return {"kind": kind, "scene": "street", "frames": frames,
            "factors": min(factors, frames * (frames - 1) // 2), "lo": pts // 4 if own else 0,
            "hi": pts if own else 0, "target": pts, "resolution": r,
            "tile": rng.choice([0, 0, 2304, 4608, 13824]),
            "layout": rng.choice(["grouped", "grouped", "interleaved", "balanced"]),
            "reorder": rng.random() < 0.3, "graph": rng.random() < 0.5, "accum": accum,
            "form": "auto" if accum == "f64" else rng.choice(["auto", "auto", "auto", "pair"])}


# ---------------------------------------------------------------- inputs

RINGS, AZIMUTHS, REACH = 64, 1024, 80.0


def _generator(seed, device="cuda"):
    return torch.Generator(device=device).manual_seed(1000003 * seed + 17)


def _rotation(axis, angle):
    x, y, z = axis / np.linalg.norm(axis)
    K = np.array([[0, -z, y], [z, 0, -x], [-y, x, 0]])
    return np.eye(3) + math.sin(angle) * K + (1 - math.cos(angle)) * (K @ K)


def _perturb(R, t, rng, trans, deg):
    """(R, t) composed on the right with a random motion of that size."""
    u = rng.normal(size=3)
    return R @ _rotation(rng.normal(size=3), math.radians(deg)), t + R @ (trans * u / np.linalg.norm(u))


def _rows(Rs, ts):
    return np.concatenate([np.asarray(Rs).reshape(-1, 9), np.asarray(ts).reshape(-1, 3)], 1)


def _covariances(normals, g):
    """xx xy xz yy yz zz of plane-like covariances (1, 1, 1e-3) about noisy normals."""
    n = normals + 0.05 * torch.randn(normals.shape, generator=g, device=normals.device)
    n = n / n.norm(dim=1, keepdim=True)
    x, y, z = n[:, 0], n[:, 1], n[:, 2]
    w = 1.0 - 1e-3
    return torch.stack([1 - w * x * x, -w * x * y, -w * x * z, 1 - w * y * y, -w * y * z,
                        1 - w * z * z], 1).contiguous()


def _room(n, g):
    """Points and normals on the floor and walls of a 40 m x 40 m x 5 m room."""
    u = torch.rand((n, 3), generator=g, device="cuda")
    which = torch.rand(n, generator=g, device="cuda")
    a, b, h = 40 * u[:, 0] - 20, 40 * u[:, 1] - 20, 5 * u[:, 2]
    side = ((which - 0.667) / 0.333 * 4).floor().clamp(0, 3)
    far = torch.where(side % 2 == 0, 20.0, -20.0)
    floor, along_x = which < 0.667, side < 2
    zero, one = torch.zeros_like(a), torch.ones_like(a)
    x = torch.where(floor, a, torch.where(along_x, far, a))
    y = torch.where(floor, b, torch.where(along_x, a, far))
    p = torch.stack([x, y, torch.where(floor, zero, h)], 1)
    nrm = torch.stack([torch.where(~floor & along_x, one, zero),
                       torch.where(~floor & ~along_x, one, zero),
                       torch.where(floor, one, zero)], 1)
    return p + 0.02 * torch.randn(p.shape, generator=g, device="cuda"), nrm


class _Street:
    """Facades at 8 to 12 m on both sides, with gaps, and poles along the x axis; scans of
    frames 1 m apart (points in ring order, in the sensor frame, with normals)."""

    def __init__(self, frames, seed, trans, deg):
        rng = np.random.default_rng([seed, 1])
        self.rng, self.frames, self.g = rng, frames, _generator(seed)
        self.walls, self.poles = [], []
        for side in (1.0, -1.0):
            x = -110.0
            while x < frames + 110.0:
                length = rng.uniform(5, 15)
                if rng.uniform() > 0.15:
                    self.walls.append((x, x + length, side * rng.uniform(8, 12), rng.uniform(10, 30)))
                x += length
        x = -110.0
        while x < frames + 110.0:
            x += rng.uniform(10, 25)
            self.poles.append((x, math.copysign(6.5, rng.uniform() - 0.5)))
        yaw = rng.uniform(-0.05, 0.05, size=frames)
        self.R = [_rotation(np.array([0.0, 0, 1]), a) for a in yaw]
        self.t = [np.array([float(f), rng.normal(0, 0.3), 1.8]) for f in range(frames)]
        est = [_perturb(R, t, rng, trans, deg) for R, t in zip(self.R, self.t)]
        self.poses = _rows([R for R, _ in est], [t for _, t in est])

    def scans(self):
        """Per frame: points (V, 3) and normals (V, 3) of the valid returns."""
        el = torch.deg2rad(torch.linspace(-25.0, 2.0, RINGS, device="cuda"))
        az = 2 * math.pi * torch.arange(AZIMUTHS, device="cuda") / AZIMUTHS
        d_s = torch.stack([(el.cos()[:, None] * az.cos()).reshape(-1),
                           (el.cos()[:, None] * az.sin()).reshape(-1),
                           el.sin()[:, None].expand(-1, AZIMUTHS).reshape(-1)], 1)
        step = 16
        for f0 in range(0, self.frames, step):
            fs = range(f0, min(f0 + step, self.frames))
            R = torch.tensor(np.stack([self.R[f] for f in fs]), dtype=torch.float32, device="cuda")
            o = torch.tensor(np.stack([self.t[f] for f in fs]), dtype=torch.float32, device="cuda")
            d = torch.matmul(d_s[None], R.transpose(1, 2).contiguous())
            dx, dy, dz = d[..., 0], d[..., 1], d[..., 2]
            ox, oy, oz = o[:, 0, None], o[:, 1, None], o[:, 2, None]
            best = torch.where(dz < -1e-6, -oz / dz.clamp(max=-1e-6), torch.inf)
            nx, ny, nz = torch.zeros_like(best), torch.zeros_like(best), torch.ones_like(best)
            for x0, x1, y, h in self.walls:
                if x1 < fs[0] - REACH or x0 > fs[-1] + REACH:
                    continue
                t = (y - oy) / dy
                x, z = ox + t * dx, oz + t * dz
                ok = (t > 0) & (x >= x0) & (x < x1) & (z >= 0) & (z <= h) & (t < best)
                best = torch.where(ok, t, best)
                ny, nz = torch.where(ok, 1.0, ny), torch.where(ok, 0.0, nz)
            a = dx * dx + dy * dy
            for px, py in self.poles:
                if px < fs[0] - REACH or px > fs[-1] + REACH:
                    continue
                bx, by = ox - px, oy - py
                b = dx * bx + dy * by
                disc = b * b - a * (bx * bx + by * by - 0.15 ** 2)
                t = (-b - disc.clamp(min=0).sqrt()) / a
                z = oz + t * dz
                ok = (disc >= 0) & (t > 0) & (z >= 0) & (z <= 6.0) & (t < best)
                best = torch.where(ok, t, best)
                nx = torch.where(ok, (bx + t * dx) / 0.15, nx)
                ny = torch.where(ok, (by + t * dy) / 0.15, ny)
                nz = torch.where(ok, 0.0, nz)
            valid = best <= REACH
            rng_m = best + 0.02 * torch.randn(best.shape, generator=self.g, device="cuda")
            nrm = torch.matmul(torch.stack([nx, ny, nz], 2), R.contiguous())
            for k in range(len(fs)):
                keep = valid[k].nonzero()[:, 0]
                yield d_s[keep] * rng_m[k, keep, None], nrm[k, keep]

    def subsample(self, scan, n):
        """n points of a scan in its order, one from each of n strata."""
        p, nrm = scan
        u = torch.rand(n, generator=self.g, device="cuda", dtype=torch.float64)
        at = (torch.arange(n, device="cuda") + u) * (p.shape[0] / n)
        at = at.long().clamp(max=p.shape[0] - 1)
        return p[at].T.contiguous(), _covariances(nrm[at], self.g)


def _pairs(frames, count, rng):
    """`count` random pairs (i, j), j < i, of frames within 20 m."""
    cand = [(i, j) for i in range(frames) for j in range(max(0, i - 20), i)]
    order = rng.permutation(len(cand))[:count]
    return [cand[k] for k in order]


def _graph_inputs(case, seed):
    """Clouds, maps' clouds, factor rows and poses of a factor graph."""
    if case.get("scene") == "room":
        g, rng = _generator(seed), np.random.default_rng([seed, 2])
        clouds = []
        for n in (case["lo"], case["target"]):
            p, nrm = _room(n, g)
            clouds.append((p.T.contiguous(), _covariances(nrm, g)))
        R, t = _perturb(np.eye(3), np.zeros(3), rng, 0.1, 2.0)
        return clouds[:1], clouds[1:], np.array([[0, 0, 0, 1]], np.int32), _rows(
            [R, np.eye(3)], [t, np.zeros(3)])
    frames = case["frames"]
    near = case["kind"] in ("iteration", "build")
    street = _Street(frames, seed, *((0.02, 0.2) if near else (0.1, 2.0)))
    own = case.get("hi", 0) > 0
    scans, targets = [], []
    for s in street.scans():
        targets.append(street.subsample(s, case["target"]))
        scans.append(s if own else None)
    if near:
        pairs = [(a, b) for a in range(frames) for b in range(a)]
    else:
        pairs = _pairs(frames, case["factors"], street.rng)
    if not own:
        return targets, targets, np.array([(i, j, i, j) for i, j in pairs], np.int32), street.poses
    size = street.rng.integers(case["lo"], case["hi"] + 1, size=len(pairs))
    sources = [street.subsample(scans[i], int(n)) for (i, _), n in zip(pairs, size)]
    rows = np.array([(k, j, i, j) for k, (i, j) in enumerate(pairs)], np.int32)
    return sources, targets, rows, street.poses


def _trial(poses, seed):
    """The poses of an optimizer's trial step, 1 cm / 0.1 degrees away."""
    rng = np.random.default_rng([seed, 3])
    out = [_perturb(p[:9].reshape(3, 3), p[9:], rng, 0.01, 0.1) for p in poses]
    return _rows([R for R, _ in out], [t for _, t in out])


def _cloud(case, seed):
    """The cloud of a voxelize case: a scan, or several merged in the first one's frame."""
    n, per = case["points"], 20000
    frames = max(1, math.ceil(n / per)) if n > 40000 else 1
    street = _Street(frames, seed, 0.0, 0.0)
    xs, cs, left = [], [], n
    for f, s in enumerate(street.scans()):
        k = math.ceil(left / (frames - f))
        left -= k
        at = torch.rand(k, generator=street.g, device="cuda", dtype=torch.float64)
        at = ((torch.arange(k, device="cuda") + at) * (s[0].shape[0] / k)).long()
        at = at.clamp(max=s[0].shape[0] - 1)
        R0, R = street.R[0], street.R[f]
        Rr = torch.tensor(R0.T @ R, dtype=torch.float32, device="cuda")
        tr = torch.tensor(R0.T @ (street.t[f] - street.t[0]), dtype=torch.float32, device="cuda")
        xs.append(s[0][at] @ Rr.T.contiguous() + tr)
        cs.append(_covariances(s[1][at] @ Rr.T.contiguous(), street.g))
    return torch.cat(xs).T.contiguous(), torch.cat(cs).contiguous()


def _serving_inputs(case, seed):
    """Host clouds of the resident keyframes, their poses and the two optimizers' requests
    (rows over frame indices, each with the poses of its own variables)."""
    street = _Street(case["frames"], seed, 0.1, 2.0)
    clouds = [street.subsample(s, case["target"]) for s in street.scans()]
    n = case["frames"]
    newest = range(n - min(case["window"], n - 1), n)
    glob = [(a, b) for a in newest for b in range(max(0, a - case["reach"]), a)]
    loc_ids = range(n - min(case["local"], n), n)
    requests = []
    for rows in (glob, [(a, b) for a in loc_ids for b in loc_ids if b < a]):
        used = sorted({k for ab in rows for k in ab})
        var = {k: v for v, k in enumerate(used)}
        requests.append((np.array([(a, b, var[a], var[b]) for a, b in rows], np.int32),
                         np.ascontiguousarray(street.poses[used]), used))
    return clouds, requests


# ---------------------------------------------------------------- the program

_shared = {}


def _context():
    """The program's one context, on a stream of its own (graph replay needs one)."""
    if not _shared:
        stream = torch.cuda.Stream()
        torch.cuda.set_stream(stream)
        _shared["ctx"] = vg.Context(0, stream=stream)
    return _shared["ctx"]


def _outputs(F):
    return {"H": torch.empty((F, 12, 12), dtype=torch.float64, device="cuda"),
            "b": torch.empty((F, 12), dtype=torch.float64, device="cuda"),
            "e": torch.empty((F,), dtype=torch.float64, device="cuda"),
            "inliers": torch.empty((F,), dtype=torch.int64, device="cuda")}


def prepare(case, seed):
    ctx = _context()
    kind = case["kind"]
    st = {"kind": kind, "ctx": ctx, "case": case}
    if kind == "voxelize":
        # the program keeps maps in arrays with room for one voxel per point
        n = case["points"]
        st["cloud"] = _cloud(case, seed)
        st["out"] = {"keys": torch.zeros((n, 3), dtype=torch.int32, device="cuda"),
                     "mean": torch.zeros((n, 3), device="cuda"),
                     "cov": torch.zeros((n, 6), device="cuda"),
                     "count": torch.zeros((n,), dtype=torch.int32, device="cuda")}
    elif kind == "connect":
        street = _Street(case["frames"], seed, 0.1, 2.0)
        clouds = [street.subsample(s, case["target"]) for s in street.scans()]
        st["maps"] = [vg.voxelize(ctx, *c, case["resolution"]) for c in clouds[:-1]]
        st["xyz"], st["poses"] = clouds[-1][0], street.poses
    elif kind == "serving":
        clouds, requests = _serving_inputs(case, seed)
        srv = vg.Server(inflight=2)
        ids = np.array([srv.add_frame(x.T.cpu().numpy(), c.cpu().numpy(), case["resolution"])
                        for x, c in clouds], np.int32)
        st["server"] = srv
        st["requests"] = [(np.concatenate([ids[rows[:, :2]], rows[:, 2:]], 1).astype(np.int32), P)
                          for rows, P, _ in requests]
        st["previous"] = [None, None]
    else:
        sources, targets, rows, poses = _graph_inputs(case, seed)
        st["poses"] = torch.from_numpy(poses).cuda()
        if kind == "build":
            st.update(clouds=targets, rows=rows)
            return st
        maps = [vg.voxelize(ctx, *c, case["resolution"]) for c in targets]
        fs = vg.FactorSet(ctx, sources, maps, rows, len(poses), case.get("tile", 0))
        st["fs"], F = fs, len(rows)
        if case.get("reorder"):
            vg.reorder_by_target(ctx, fs, st["poses"])
        if case.get("layout", "grouped") != "grouped":
            vg.set_layout(ctx, fs, case["layout"])
        if kind == "cost":
            st["out"] = {k: v for k, v in _outputs(F).items() if k in ("e", "inliers")}
        elif kind == "overlap":
            st["out"] = {"hits": torch.empty((F,), dtype=torch.int64, device="cuda"),
                         "overlap": torch.empty((F,), dtype=torch.float64, device="cuda")}
        else:
            st["out"] = _outputs(F)
        if kind == "iteration":
            P, K = len(poses), fs.pairs.shape[0]
            st["trial"] = torch.from_numpy(_trial(poses, seed)).cuda()
            st["system"] = {
                "Hdiag": torch.empty((P, 6, 6), dtype=torch.float64, device="cuda"),
                "bvec": torch.empty((P, 6), dtype=torch.float64, device="cuda"),
                "Hoff": torch.empty((K, 6, 6), dtype=torch.float64, device="cuda")}
            st["trial_out"] = {k: v for k, v in _outputs(F).items() if k in ("e", "inliers")}
    return st


def run(st):
    kind, ctx = st["kind"], st["ctx"]
    if kind == "round":
        c = st["case"]
        return vg.linearize_factors(ctx, st["fs"], st["poses"], accum=c["accum"],
                                    use_graph=c["graph"], form=c["form"], out=st["out"])
    if kind == "cost":
        return vg.evaluate_errors(ctx, st["fs"], st["poses"], out=st["out"])
    if kind == "overlap":
        return vg.overlap(ctx, st["fs"], st["poses"], out=st["out"])
    if kind == "iteration":
        out = vg.linearize_factors(ctx, st["fs"], st["poses"], out=st["out"])
        system = vg.assemble_system(ctx, st["fs"], out["H"], out["b"], out=st["system"])
        trial = vg.evaluate_errors(ctx, st["fs"], st["trial"], out=st["trial_out"])
        return {"factors": out, "system": system, "trial": trial}
    if kind == "build":
        maps = [vg.voxelize(ctx, *c, st["case"]["resolution"]) for c in st["clouds"]]
        fs = vg.FactorSet(ctx, st["clouds"], maps, st["rows"], st["poses"].shape[0])
        return vg.linearize_factors(ctx, fs, st["poses"])
    if kind == "voxelize":
        vmap = vg.voxelize(ctx, *st["cloud"], st["case"]["resolution"])
        out = st["out"]
        if vg.lib().vgicp_map_export(ctx.handle, vmap.handle, out["keys"].data_ptr(),
                                     out["mean"].data_ptr(), out["cov"].data_ptr(),
                                     out["count"].data_ptr()) != vg.OK:
            raise RuntimeError("vgicp_map_export failed")
        return out
    if kind == "connect":
        return vg.connect(ctx, st["xyz"], st["poses"][-1], st["maps"], st["poses"][:-1],
                          threshold=0.05, rule="at_least")
    st["previous"] = [st["server"].submit("linearize", rows, P, out=prev)
                      for (rows, P), prev in zip(st["requests"], st["previous"])]
    return [{"H": r.H, "b": r.b, "e": r.e, "inliers": r.inliers}
            for r in (q.wait() for q in st["previous"])]


# ---------------------------------------------------------------- work

def work(case):
    """Each point, hit covariance, touched voxel and result moved once: 40 % of a graph's points
    fall in a voxel, three quarters for frames of one submap; a hit takes about 450 operations,
    a lookup 30."""
    kind = case["kind"]
    if kind == "voxelize":
        n = case["points"]
        return {"bytes": 36 * n + 52 * n / 4, "flops": 12 * n}
    n, hit = case["target"], 0.4
    if kind == "connect":
        pts = n * (case["frames"] - 1)
        return {"bytes": 12 * n + 9 * n / 4 * (case["frames"] - 1), "flops": 30 * pts}
    if kind == "serving":
        F = (min(case["window"], case["frames"] - 1) * min(case["reach"], case["frames"] - 1)
             + case["local"] * (case["local"] - 1) // 2)
    elif kind in ("iteration", "build"):
        F, hit = case["frames"] * (case["frames"] - 1) // 2, 0.75
    else:
        F = case["factors"]
    if case.get("hi"):
        n = (case["lo"] + case["hi"]) / 2
    pts = F * n
    if kind == "overlap":
        return {"bytes": 12 * pts + 9 * pts / 20, "flops": 30 * pts}
    per_round = 12 * pts + 24 * hit * pts + 44 * hit * pts / 8
    flops = (30 + 450 * hit) * pts
    if kind == "cost":
        return {"bytes": per_round + 16 * F, "flops": 0.6 * flops}
    extra = 0
    if kind == "iteration":
        extra, flops = per_round + 16 * F + 2 * 156 * 8 * F, 1.6 * flops
    if kind == "build":
        extra = 2 * 88 * case["frames"] * case["target"]
    return {"bytes": per_round + 158 * 8 * F + extra, "flops": flops}


# ---------------------------------------------------------------- 64 bits

def _full(c):
    i = [0, 1, 2, 1, 3, 4, 2, 4, 5]
    return c.double()[:, i].reshape(-1, 3, 3)


def _scale(resolution):
    return float(np.float32(1.0 / resolution))


def _map64(cloud, resolution):
    """Voxels in key order: packed keys, FP64 means and covariances."""
    x, c = cloud
    s = torch.tensor(_scale(resolution), dtype=torch.float32, device="cuda")
    k = (x * s).floor().long() + (1 << 20)
    packed = (k[0] << 42) | (k[1] << 21) | k[2]
    keys, inv, count = torch.unique(packed, return_inverse=True, return_counts=True)
    V = keys.shape[0]
    mean = torch.zeros((V, 3), dtype=torch.float64, device="cuda").index_add_(0, inv, x.T.double())
    cov = torch.zeros((V, 6), dtype=torch.float64, device="cuda").index_add_(0, inv, c.double())
    return keys, mean / count[:, None], cov / count[:, None]


def _stored(m):
    """A map as factors read it: means and covariances rounded to FP32."""
    return m[0], m[1].float(), m[2].float()


def _relative(pi, pj):
    Ri, Rj = pi[:9].reshape(3, 3), pj[:9].reshape(3, 3)
    return Rj.T @ Ri, Rj.T @ (pi[9:] - pj[9:])


def _lookup64(x, m, R, t, resolution):
    """Voxel of each point (or -1): FP32 coordinates by fused multiply-adds."""
    s = _scale(resolution)
    S = torch.from_numpy((s * R).astype(np.float32)).cuda().double()
    u = torch.from_numpy((s * t).astype(np.float32)).cuda().double()
    p = x.double()
    v = u[:, None].expand(3, x.shape[1])
    for a in range(3):
        v = (S[:, a, None] * p[a] + v).float().double()
    k = v.floor().long() + (1 << 20)
    want = (k[0] << 42) | (k[1] << 21) | k[2]
    at = torch.searchsorted(m[0], want).clamp(max=m[0].shape[0] - 1)
    return torch.where(m[0][at] == want, at, -1)


def _skew(v):
    z = torch.zeros_like(v[:, 0])
    return torch.stack([z, -v[:, 2], v[:, 1], v[:, 2], z, -v[:, 0], -v[:, 1], v[:, 0], z],
                       1).reshape(-1, 3, 3)


def _dot(A, B):
    """Products of (n, a, 3) and (n, 3, b) stacks, entry by entry."""
    return (A[:, :, :, None] * B[:, None, :, :]).sum(2)


def _factor64(cloud, m, pi, pj, resolution, hessian=True):
    """H, b, e of one factor."""
    R, t = _relative(pi, pj)
    at = _lookup64(cloud[0], m, R, t, resolution)
    hit = (at >= 0).nonzero()[:, 0]
    at = at[hit]
    Rg, tg = torch.from_numpy(R).cuda(), torch.from_numpy(t).cuda()
    n = hit.shape[0]
    mu = cloud[0].double().T[hit]
    q = mu @ Rg.T.contiguous() + tg
    Rn = Rg[None].expand(n, 3, 3)
    RC = _dot(Rn, _full(cloud[1][hit]))
    F = _full(m[2][at]) + _dot(RC, Rn.transpose(1, 2))
    c = torch.stack([torch.linalg.cross(F[:, 1], F[:, 2]), torch.linalg.cross(F[:, 2], F[:, 0]),
                     torch.linalg.cross(F[:, 0], F[:, 1])], 2)
    W = c / (F[:, 0] * c[:, :, 0]).sum(1)[:, None, None]
    d = m[1][at].double() - q
    Wd = (W * d[:, None, :]).sum(2)
    e = (d * Wd).sum()
    if not hessian:
        return None, None, e
    J = torch.cat([_dot(Rn, _skew(mu)), -Rn, -_skew(q),
                   torch.eye(3, dtype=torch.float64, device="cuda")[None].expand(n, 3, 3)], 2)
    WJ = _dot(W, J)
    H = J.reshape(-1, 12).T.contiguous() @ WJ.reshape(-1, 12)
    return H, (J * Wd[:, :, None]).sum((0, 1)), e


def _factors64(sources, maps, rows, poses, resolution, hessian=True):
    out = [_factor64(sources[s], maps[m], poses[i], poses[j], resolution, hessian)
           for s, m, i, j in rows]
    e = torch.stack([o[2] for o in out])
    if not hessian:
        return {"e": e, "inliers": None}
    return {"H": torch.stack([o[0] for o in out]), "b": torch.stack([o[1] for o in out]),
            "e": e, "inliers": None}


def exact(case, seed):
    kind, r = case["kind"], case["resolution"]
    if kind == "voxelize":
        _, mean, cov = _map64(_cloud(case, seed), r)
        pad = (0, 0, 0, case["points"] - mean.shape[0])
        mean, cov = (torch.nn.functional.pad(v, pad) for v in (mean, cov))
        return {"keys": None, "mean": mean, "cov": cov, "count": None}
    if kind == "connect":
        street = _Street(case["frames"], seed, 0.1, 2.0)
        clouds = [street.subsample(s, case["target"]) for s in street.scans()]
        x, P = clouds[-1][0], street.poses
        hits = [(_lookup64(x, _map64(c, r), *_relative(P[-1], P[k]), r) >= 0).sum()
                for k, c in enumerate(clouds[:-1])]
        return {"hits": None, "overlap": torch.stack(hits).double() / x.shape[1],
                "admitted": None}
    if kind == "serving":
        clouds, requests = _serving_inputs(case, seed)
        maps = [_stored(_map64(c, r)) for c in clouds]
        return [_factors64(clouds, maps, rows, P, r) for rows, P, _ in requests]
    sources, targets, rows, poses = _graph_inputs(case, seed)
    maps = [_stored(_map64(c, r)) for c in targets]
    if kind == "cost":
        return _factors64(sources, maps, rows, poses, r, hessian=False)
    if kind == "overlap":
        hits = [(_lookup64(sources[s][0], maps[m], *_relative(poses[i], poses[j]), r) >= 0).sum()
                for s, m, i, j in rows]
        return {"hits": None, "overlap": torch.stack(hits).double() / case["target"]}
    out = _factors64(sources, maps, rows, poses, r)
    if kind != "iteration":
        return out
    P = len(poses)
    pairs = sorted({(min(i, j), max(i, j)) for _, _, i, j in rows})
    Hd = torch.zeros((P, 6, 6), dtype=torch.float64, device="cuda")
    bv = torch.zeros((P, 6), dtype=torch.float64, device="cuda")
    Ho = torch.zeros((len(pairs), 6, 6), dtype=torch.float64, device="cuda")
    for f, (_, _, i, j) in enumerate(rows):
        H, b = out["H"][f], out["b"][f]
        Hd[i] += H[:6, :6]
        Hd[j] += H[6:, 6:]
        bv[i] += b[:6]
        bv[j] += b[6:]
        Ho[pairs.index((min(i, j), max(i, j)))] += H[:6, 6:] if i < j else H[6:, :6]
    return {"factors": out, "system": {"Hdiag": Hd, "bvec": bv, "Hoff": Ho},
            "trial": _factors64(sources, maps, rows, _trial(poses, seed), r, hessian=False)}

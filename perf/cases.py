"""Performance cases: the calls that a user of the library makes, over the sizes that they are made at.

A case names one public entry point and the sizes of its inputs.  Inputs are ray-cast LiDAR scans (spinning sensor,
ground plane, car-sized boxes, ego motion between sweeps), made on the GPU with torch from the seed; `exact` is the
definition of the entry points in include/mmbev.h, in plain torch.
"""
import math
import types

import numpy as np
import torch

from paper_2608_15437_amd import mmbev

DEV = "cuda"

# ------------------------------------------------------------------ the cases

_NUSC = dict(beams=32, azimuths=1085, sweeps=10, elev_lo=-30.0, elev_hi=10.0, height=1.8, obstacles=30, obs_far=50.0,
             features=5, on=30, extra=2, random=0, extent=54.0, margin=0.5, budget_lo=1, budget_hi=10, cover=False,
             xy=54.0, z_lo=-5.0, voxel=0.075, voxel_z=0.2, dx=1440, dy=1440, dz=40, max_points=10, max_voxels=120000,
             rate=0.0, ragged=False, pad=0, noalloc=False, kept=0.06, voxels=0.02)
_OUSTER = dict(_NUSC, beams=128, azimuths=1024, sweeps=3, elev_lo=-22.5, elev_hi=22.5, height=1.0, obstacles=40,
               obs_far=38.0, on=40, extra=0, random=24, extent=40.0, margin=0.3, budget_hi=3, xy=40.0, z_lo=-3.0,
               voxel=0.05, voxel_z=0.15, dx=1600, dy=1600, max_points=8, max_voxels=200000, kept=0.19, voxels=0.047)


def listed():
    return [
        # One sweep of a small sensor with four regions of interest: the smallest call, launches and latency alone.
        dict(_NUSC, name="vox_small", kind="voxelize", frames=1, azimuths=625, sweeps=1, obstacles=6, features=4, on=0,
             extra=0, random=4, extent=30.0, budget_hi=1, xy=51.2, voxel=0.2, dx=512, dy=512, max_voxels=20000,
             kept=0.003, voxels=0.003),
        # One ten-sweep nuScenes-shaped frame inside its tracked objects' regions: the call of every detection frame.
        dict(_NUSC, name="vox_frame", kind="voxelize", frames=1),
        # The same frame with one region over everything (a keyframe): most points are kept and the voxel cap binds.
        dict(_NUSC, name="vox_keyframe", kind="voxelize", frames=1, obstacles=30, on=0, extra=0, cover=True,
             budget_lo=10, kept=0.72, voxels=0.345),
        # A three-sweep 128-beam robot frame with 64 regions, through the entry point of serving loops that allocate
        # nothing.
        dict(_OUSTER, name="vox_robot", kind="voxelize", frames=1, noalloc=True),
        # Eight frames with 256 overlapping regions each on a 0.05 m grid: crowded scenes.
        dict(_NUSC, name="vox_crowded", kind="voxelize", frames=8, random=226, extra=0, voxel=0.05, dx=2160, dy=2160,
             max_voxels=160000, kept=0.13, voxels=0.077),
        # 128 nuScenes-shaped frames in one call: offline processing of a log, the largest input.
        dict(_NUSC, name="vox_batch", kind="voxelize", frames=128),
        # Five frames of odd, unequal sizes with padded feature rows, a tenth of the points outside the regions kept
        # (the background keep rate of training and keyframe refresh).
        dict(_NUSC, name="vox_background", kind="voxelize", frames=5, features=4, max_points=5, rate=0.1, ragged=True,
             pad=37, kept=0.13, voxels=0.11),
        # Pillar map of one frame, and the whole voxel grid's map of one frame: the dense input of a BEV backbone.
        dict(_NUSC, name="bev_pillars", kind="bev", frames=1, voxel=0.2, voxel_z=8.0, dx=512, dy=512, dz=1, xy=51.2,
             max_points=20, max_voxels=30000),
        dict(_NUSC, name="bev_grid", kind="bev", frames=1),
        # Object clusters of one robot frame, and of 128 frames of a log.
        dict(_OUSTER, name="clusters_robot", kind="clusters", frames=1, layer=12, shift=0, neighbours=8, least=2),
        dict(_NUSC, name="clusters_batch", kind="clusters", frames=128, layer=18, shift=0, neighbours=8, least=2),
        # Regions and sweep budgets of 128 frames from the detections of the frames before (host code).
        dict(name="selector", kind="selector", frames=128, detections=64),
    ]


def draw(rng):
    """One more case of the same ranges: frames of one to ten sweeps, odd ray counts, one frame to a long batch."""
    def spread(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["voxelize"] * 6 + ["bev", "clusters", "selector"])
    if kind == "selector":
        return dict(kind=kind, frames=spread(4, 128), detections=rng.randint(8, 64))
    c = dict(_OUSTER if rng.random() < 0.25 else _NUSC, kind=kind)
    c["sweeps"] = rng.randint(1, c["sweeps"])
    c["azimuths"] = rng.randint(500, c["azimuths"])
    c["frames"] = spread(1, 128 if c["beams"] == 32 else 32)
    c["budget_hi"] = c["sweeps"]
    c["random"] = rng.choice([0, 0, 7, 34, 90, 226])
    c["kept"], c["voxels"] = (0.06, 0.02) if c["random"] < 30 else (0.13, 0.07)
    c["features"] = rng.randint(3, 6)
    c["max_points"] = rng.randint(4, 12)
    if kind == "voxelize":
        style = rng.random()
        c["ragged"] = rng.random() < 0.4
        c["pad"] = rng.choice([0, 0, 3, 64])
        if style < 0.15:
            c.update(cover=True, on=0, extra=0, random=0, budget_lo=c["sweeps"], frames=min(c["frames"], 8), kept=0.72,
                     voxels=0.35)
        elif style < 0.35:
            c.update(rate=rng.choice([0.01, 0.05, 0.1]), frames=min(c["frames"], 24), kept=0.15, voxels=0.1)
        if rng.random() < 0.3:
            c.update(voxel=0.1, dx=int(c["xy"] * 20), dy=int(c["xy"] * 20))
    elif kind == "bev":
        c.update(frames=1, dx=rng.randint(700, 1440), dz=rng.randint(1, 40), features=rng.randint(3, 5))
    else:
        c.update(frames=min(c["frames"], 96), layer=rng.randint(10, 20), shift=rng.randint(0, 2),
                 neighbours=rng.choice([4, 8]), least=rng.randint(1, 3))
    return c


def _frame_sizes(c):
    """Points of each frame; unequal and odd ones where the case is ragged (rays without a return are left out)."""
    full = c["sweeps"] * c["beams"] * c["azimuths"]
    if not c["ragged"]:
        return [full] * c["frames"]
    return [int(full * (0.55 + 0.45 * math.modf((f + 1) * 0.6180339887)[0])) | 1 for f in range(c["frames"])]


def _rois_of(c):
    return 1 if c["cover"] else c["on"] + c["extra"] + c["random"]


def work(c):
    """Every input read once, every output written once; kept points and voxels from the usual share of the points."""
    if c["kind"] == "selector":
        n = c["frames"] * c["detections"]
        return {"bytes": n * (64 + 2 * 33 + 16) + c["frames"] * 40, "flops": n * 150}
    n, b = sum(_frame_sizes(c)), c["frames"]
    rows = min(c["voxels"] * n, b * c["max_voxels"])
    if c["kind"] == "bev":
        return {"bytes": 4 * b * c["features"] * c["dx"] * c["dy"] * c["dz"] + rows * (16 + 4 * c["features"]),
                "flops": 0}
    if c["kind"] == "clusters":
        return {"bytes": rows * (16 + 4 + 4), "flops": rows * 20}
    row = 16 + 4 + 4 * c["features"] + 4 * c["max_points"]
    return {"bytes": 13 * n + 4 * (c["features"] - 3) * c["kept"] * n + row * rows + b * (33 * _rois_of(c) +
                                                                                         48 * c["sweeps"]),
            "flops": 35 * n}


def tolerance(c):
    """Voxels, counts, point indices and their order are whole numbers and unique.  Means are sums in 64 bits rounded
    once to 32: sums in another order move few of them by one unit in the last place.  A map holds copies."""
    if c["kind"] in ("bev", "clusters"):
        return "exact"
    return {"rel": 1e-7, "max": 5e-7, "differ": 0.0}


# ------------------------------------------------------------------ the inputs

def _obstacles(c, rng):
    """Boxes (cx, cy, cz, length, width, height, yaw) that do not overlap, the sensor's column clear."""
    got = np.zeros((0, 7))
    for _ in range(4000):
        if len(got) == c["obstacles"]:
            break
        size = np.array([4.5, 1.9, 1.7]) * rng.uniform(0.9, 1.1, 3)
        rad, az = math.sqrt(rng.uniform(9.0, c["obs_far"] ** 2)), rng.uniform(0, 2 * math.pi)
        x, y, br = rad * math.cos(az), rad * math.sin(az), 0.5 * math.hypot(size[0], size[1])
        gap = np.hypot(got[:, 0] - x, got[:, 1] - y) - 0.5 * np.hypot(got[:, 3], got[:, 4]) - br
        if rad > br + 1.0 and (len(got) == 0 or gap.min() > 0.5):
            got = np.vstack([got, [x, y, size[2] / 2, *size, rng.uniform(0, 2 * math.pi)]])
    return got


def _regions(c, obs, rng):
    """ROI descriptors (cx, cy, length, width, yaw, margin) and sweep budgets of one frame."""
    if c["cover"]:
        return np.array([[0.0, 0.0, 2.2 * c["xy"], 2.2 * c["xy"], 0.0, 0.0]]), np.array([c["budget_hi"]], np.uint8)
    on = obs[rng.integers(0, len(obs), c["on"])] if c["on"] > len(obs) else obs[:c["on"]]
    rows = [[o[0], o[1], o[3], o[4], o[6], c["margin"]] for o in on]
    rows += [[o[0] + 2.5 * math.cos(o[6]), o[1] + 2.5 * math.sin(o[6]), o[3], o[4], o[6], c["margin"]]
             for o in obs[:c["extra"]]]
    for k in range(c["random"]):
        x, y = rng.uniform(-c["extent"], c["extent"], 2)
        if k % 5 == 4 and rows:  # every fifth one over an earlier one
            e = rows[rng.integers(0, len(rows))]
            x, y = e[0] + rng.uniform(-2, 2), e[1] + rng.uniform(-2, 2)
        rows.append([x, y, 4.5 * rng.uniform(0.9, 1.1), 1.9 * rng.uniform(0.9, 1.1), rng.uniform(0, 2 * math.pi),
                     c["margin"]])
    return np.array(rows), rng.integers(c["budget_lo"], c["budget_hi"] + 1, len(rows)).astype(np.uint8)


def _scan(c, obs, rng, gen):
    """One frame's points [C][n], sweep ids and poses [S][12]: rays cast from each sweep's own pose."""
    S, nb, na = c["sweeps"], c["beams"], c["azimuths"]
    speed, turn = rng.uniform(0, 15), rng.uniform(-0.3, 0.3)
    tau = -0.05 * np.arange(S)
    psi = turn * tau
    px = speed * tau if abs(turn) < 1e-9 else speed / turn * np.sin(turn * tau)
    py = 0 * tau if abs(turn) < 1e-9 else speed / turn * (1 - np.cos(turn * tau))
    poses = np.zeros((S, 12), np.float32)
    poses[:, 0] = poses[:, 5] = np.cos(psi)
    poses[:, 1], poses[:, 4] = -np.sin(psi), np.sin(psi)
    poses[:, 3], poses[:, 7], poses[:, 10] = px, py, 1.0
    f32 = dict(dtype=torch.float32, device=DEV)
    phase = torch.as_tensor(rng.uniform(0, 2 * math.pi / na, S), **f32).view(S, 1, 1)
    el = torch.linspace(c["elev_lo"] * math.pi / 180, c["elev_hi"] * math.pi / 180, nb, **f32).view(1, nb, 1)
    az = phase + torch.arange(na, **f32).view(1, 1, na) * (2 * math.pi / na)
    d = [(torch.cos(el) * torch.cos(az)).reshape(S, -1), (torch.cos(el) * torch.sin(az)).reshape(S, -1),
         torch.sin(el).expand(S, nb, na).reshape(S, -1)]
    t = torch.where(d[2] < -1e-6, -c["height"] / d[2], torch.full_like(d[2], 1e9))
    for o in obs:  # slab test of every ray against the box, in the box's axes
        yaw = o[6] - psi
        col = lambda v: torch.as_tensor(v, **f32).view(S, 1)  # noqa: E731
        sx, sy = np.cos(psi) * (o[0] - px) + np.sin(psi) * (o[1] - py), -np.sin(psi) * (o[0] - px) + np.cos(psi) * (o[1] - py)
        co, si = np.cos(yaw), np.sin(yaw)
        from_, along = [col(-co * sx - si * sy), col(si * sx - co * sy), c["height"] - o[2]], [
            col(co) * d[0] + col(si) * d[1], col(co) * d[1] - col(si) * d[0], d[2]]
        lo, hi = torch.full_like(t, -1e9), torch.full_like(t, 1e9)
        for p, v, h in zip(from_, along, o[3:6] / 2):
            v = torch.where(v.abs() < 1e-7, torch.full_like(v, 1e-7), v)
            a, b = (-h - p) / v, (h - p) / v
            lo, hi = torch.maximum(lo, torch.minimum(a, b)), torch.minimum(hi, torch.maximum(a, b))
        t = torch.where((lo <= hi) & (lo > 0) & (lo < t), lo, t)
    noise = 0.02 * torch.randn(t.shape, generator=gen, **f32)
    r = torch.where(t > 100.0, torch.full_like(t, 100.0), (t + noise).clamp_min(0.05))
    feat = torch.empty((c["features"], S * nb * na), **f32)
    feat[0], feat[1], feat[2] = (r * d[0]).view(-1), (r * d[1]).view(-1), (c["height"] + r * d[2]).view(-1)
    ids = torch.arange(S, dtype=torch.uint8, device=DEV).repeat_interleave(nb * na)
    if c["features"] > 3:
        feat[3] = 255 * torch.rand(S * nb * na, generator=gen, **f32)
    if c["features"] > 4:
        feat[4] = ids.float() * 0.05
    for k in range(5, c["features"]):
        feat[k] = torch.randn(S * nb * na, generator=gen, **f32)
    return feat, ids, poses


def _inputs(c, seed):
    """The arrays of a voxelisation call, on the GPU."""
    sizes = _frame_sizes(c)
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    n = int(off[-1])
    s = types.SimpleNamespace(case=c, n=n, sizes=sizes)
    s.rows = torch.zeros((c["features"], n + c["pad"]), dtype=torch.float32, device=DEV)
    s.feat = s.rows[:, :n]
    s.ids = torch.empty(n, dtype=torch.uint8, device=DEV)
    poses, desc, budgets, roi_off = [], [], [], [0]
    for f in range(c["frames"]):
        rng = np.random.default_rng([seed, f])
        gen = torch.Generator(DEV).manual_seed((seed * 1000003 + f) % (1 << 62))
        obs = _obstacles(c, rng)
        feat, ids, pose = _scan(c, obs, rng, gen)
        if c["ragged"]:
            at = torch.randperm(feat.shape[1], generator=gen, device=DEV)[:sizes[f]].sort().values
            feat, ids = feat[:, at], ids[at]
        s.feat[:, off[f]:off[f + 1]], s.ids[off[f]:off[f + 1]] = feat, ids
        rows, bud = _regions(c, obs, rng)
        poses.append(pose)
        desc.append(rows)
        budgets.append(bud)
        roi_off.append(roi_off[-1] + len(rows))
    s.desc, s.budgets_host, s.roi_off_host = np.concatenate(desc), np.concatenate(budgets), np.array(roi_off, np.int32)
    s.offsets = torch.from_numpy(off).to(DEV)
    s.poses = torch.from_numpy(np.stack(poses)).to(DEV)
    s.budgets = torch.from_numpy(s.budgets_host).to(DEV)
    s.roi_off = torch.from_numpy(s.roi_off_host).to(DEV)
    return s


def _grid(c):
    return mmbev.grid_params((-c["xy"], -c["xy"], c["z_lo"]), (c["voxel"], c["voxel"], c["voxel_z"]),
                             (c["dx"], c["dy"], c["dz"]), c["max_points"], c["max_voxels"], c["sweeps"], c["frames"])


def _detections(c, seed):
    """Detection caches: a third of the objects ahead, the rest around; people, vehicles, static objects."""
    rng, b, n = np.random.default_rng([seed, 7]), c["frames"], c["frames"] * c["detections"]
    d = np.zeros(n, mmbev.DETECTION_DTYPE)
    ahead = rng.random(n) < 1 / 3
    d["x"] = np.where(ahead, rng.uniform(0, 45, n), rng.uniform(-60, 60, n))
    d["y"] = np.where(ahead, rng.uniform(-1, 1, n) * (0.6 * d["x"] + 2), rng.uniform(-60, 60, n))
    d["cls"] = rng.choice(3, n, p=[0.3, 0.5, 0.2])
    heading = np.where(d["cls"] == 0, rng.uniform(-np.pi, np.pi, n),
                       rng.uniform(-0.35, 0.35, n) + np.pi * (rng.random(n) < 0.25))
    speed = np.choose(d["cls"], [rng.uniform(0, 2, n), rng.uniform(0, 15, n), np.zeros(n)])
    d["yaw"], d["vx"], d["vy"] = heading, speed * np.cos(heading), speed * np.sin(heading)
    d["length"] = np.choose(d["cls"], [0.8, 4.5 * rng.uniform(0.9, 1.1, n), 0.5])
    d["width"] = np.choose(d["cls"], [0.8, 1.9 * rng.uniform(0.9, 1.1, n), 0.5])
    ego = np.zeros(b, mmbev.EGO_DTYPE)
    ego["speed"], ego["dyaw"] = rng.uniform(0, 35, b), rng.uniform(-0.15, 0.15, b)
    ego["dx"], ego["dy"] = -0.5 * ego["speed"] * np.cos(ego["dyaw"]), -0.5 * ego["speed"] * np.sin(ego["dyaw"])
    return d, (np.arange(b + 1) * c["detections"]).astype(np.int32), ego


def prepare(c, seed):
    if c["kind"] == "selector":
        d, off, ego = _detections(c, seed)
        return types.SimpleNamespace(case=c, dets=d, det_off=off, ego=ego, policy=mmbev.policy())
    s = _inputs(c, seed)
    s.grid = _grid(c)
    rows = c["frames"] * c["max_voxels"]
    i32 = dict(dtype=torch.int32, device=DEV)
    if c["kind"] == "voxelize":
        s.rois = torch.from_numpy(mmbev.make_rois(s.desc).view(np.float32).reshape(-1, 8)).to(DEV)
        s.max_rois = _rois_of(c)
        s.coords, s.counts = torch.full((rows, 4), -7, **i32), torch.full((rows,), -7, **i32)
        s.means = torch.full((rows, c["features"]), -7.0, dtype=torch.float32, device=DEV)
        s.index = torch.full((rows, c["max_points"]), -7, **i32)
        s.voxel_off = torch.zeros(c["frames"] + 1, dtype=torch.int64, device=DEV)
        if not c["noalloc"]:
            size = mmbev.roi_voxelize_workspace_bytes(s.grid, s.n, c["features"], s.max_rois)
            s.workspace = torch.empty(size, dtype=torch.uint8, device=DEV)
            mmbev.workspace_init(s.workspace)
        return s
    coords, counts, means, _, voxel_off = _voxels(s)
    n = len(coords)
    s.coords, s.counts = torch.zeros((rows, 4), **i32), torch.zeros((rows,), **i32)
    s.means = torch.zeros((rows, c["features"]), dtype=torch.float32, device=DEV)
    s.coords[:n], s.counts[:n], s.means[:n], s.voxel_off = coords.int(), counts.int(), means.float(), voxel_off
    del s.rows, s.feat
    if c["kind"] == "bev":
        s.map = torch.empty(mmbev.bev_map_shape(s.grid, c["features"]), dtype=torch.float32, device=DEV)
        return s
    params = mmbev.cluster_params(c["layer"], c["dz"], c["shift"], c["neighbours"], c["least"])
    s.proposer = mmbev.ClusterProposer(s.grid, params, DEV)
    return s


def run(s):
    c = s.case
    if c["kind"] == "selector":
        r = mmbev.build_rois(s.dets, s.det_off, s.ego, s.policy)
        return [r["rois"].view(np.float32).reshape(-1, 8), r["budgets"], r["roi_offsets"],
                np.ascontiguousarray(r["crit"]["ttc"]), np.ascontiguousarray(r["crit"]["flags"]),
                np.ascontiguousarray(r["crit"]["rank"]), r["sweeps"]]
    if c["kind"] == "bev":
        mmbev.scatter_to_bev(s.coords, s.means, s.voxel_off, s.grid, s.map)
        return s.map
    if c["kind"] == "clusters":
        s.proposer.run(s.coords, s.counts, s.voxel_off)
        return [s.proposer.out, s.proposer.offsets, s.proposer.labels]
    if c["noalloc"]:
        mmbev.roi_voxelize_noalloc(s.feat, s.offsets, s.ids, s.poses, s.rois, s.roi_off, s.budgets, s.grid, s.coords,
                                   s.counts, s.means, s.index, s.voxel_off, s.max_rois)
    else:
        mmbev.roi_voxelize(s.feat, s.offsets, s.ids, s.poses, s.rois, s.roi_off, s.budgets, s.grid, s.coords, s.counts,
                           s.means, s.index, s.voxel_off, s.workspace, s.max_rois, rho_out=c["rate"],
                           seed=1234 if c["rate"] else 0)
    return [s.coords, s.counts, s.means, s.index, s.voxel_off]


# ------------------------------------------------------------------ the definition, in 64 bits

def _fma(a, b, c):
    """A fused multiply-add of 32-bit values (their product is exact in 64 bits)."""
    return (a.double() * b.double() + c.double()).float()


def _drawn(n, rate, seed):
    """Points kept outside the regions: the SplitMix64 output of each point's index against the rate."""
    wrap = lambda v: v - (1 << 64) if v >= 1 << 63 else v  # noqa: E731
    shr = lambda z, k: (z >> k) & ((1 << (64 - k)) - 1)  # noqa: E731
    z = torch.arange(1, n + 1, dtype=torch.int64, device=DEV) * wrap(0x9E3779B97F4A7C15) + wrap(seed)
    z = (z ^ shr(z, 30)) * wrap(0xBF58476D1CE4E5B9)
    z = (z ^ shr(z, 27)) * wrap(0x94D049BB133111EB)
    return shr(z ^ shr(z, 31), 40) < round(float(np.float32(rate)) * (1 << 24))


def _voxels(s):
    """coords, counts, means (64 bits), point indices and frame offsets of the voxels of one call's inputs."""
    c, at, out, off = s.case, 0, [], [0]
    # ROI records as mmbev_make_rois defines them
    rec = np.stack([s.desc[:, 0], s.desc[:, 1], np.cos(s.desc[:, 4]), np.sin(s.desc[:, 4]),
                    s.desc[:, 2] / 2 + s.desc[:, 5], s.desc[:, 3] / 2 + s.desc[:, 5]], 1).astype(np.float32)
    low = np.array([-c["xy"], -c["xy"], c["z_lo"]], np.float32)
    size = np.array([c["voxel"], c["voxel"], c["voxel_z"]], np.float32)
    dims = (c["dx"], c["dy"], c["dz"])
    background = _drawn(s.n, c["rate"], 1234) if c["rate"] else None
    M = c["max_points"]
    for f, n in enumerate(s.sizes):
        x = s.feat[:, at:at + n]
        sweep = s.ids[at:at + n].long()
        P = s.poses[f][sweep]
        p = [_fma(P[:, 4 * d], x[0], _fma(P[:, 4 * d + 1], x[1], _fma(P[:, 4 * d + 2], x[2], P[:, 4 * d + 3])))
             for d in range(3)]
        keep = torch.zeros(n, dtype=torch.bool, device=DEV)
        for j in range(s.roi_off_host[f], s.roi_off_host[f + 1]):
            cx, cy, co, si, ex, ey = (torch.tensor(v, device=DEV) for v in rec[j])
            dx, dy = p[0] - cx, p[1] - cy
            lx, ly = _fma(co, dx, si * dy), _fma(co, dy, -(si * dx))
            keep |= (sweep < int(s.budgets_host[j])) & (lx.abs() <= ex) & (ly.abs() <= ey)
        if background is not None:
            keep |= background[at:at + n]
        cell = []
        for d in range(3):
            q = ((p[d] - torch.tensor(low[d], device=DEV)).double() / float(size[d])).float()
            keep &= (q >= 0) & (q < dims[d])
            cell.append(q)
        k = keep.nonzero().view(-1)
        ix, iy, iz = (q[k].long() for q in cell)
        key, order = ((iz * dims[1] + iy) * dims[0] + ix).sort(stable=True)
        k = k[order]
        uniq, number, count = torch.unique_consecutive(key, return_inverse=True, return_counts=True)
        start = count.cumsum(0) - count
        if len(uniq) > c["max_voxels"]:  # the voxels whose first point comes first
            chosen = torch.zeros(len(uniq), dtype=torch.bool, device=DEV)
            chosen[k[start].sort().indices[:c["max_voxels"]]] = True
        else:
            chosen = torch.ones(len(uniq), dtype=torch.bool, device=DEV)
        rank = torch.arange(len(k), device=DEV) - start[number]
        use = (rank < M) & chosen[number]
        row = (chosen.cumsum(0) - 1)[number][use]
        V = int(chosen.sum())
        index = torch.full((V, M), -1, dtype=torch.int64, device=DEV)
        index[row, rank[use]] = k[use] + at
        count = count[chosen].clamp_max(M)
        means = torch.zeros((V, c["features"]), dtype=torch.float64, device=DEV)
        for d in range(c["features"]):
            v = (p[d] if d < 3 else x[d])[k[use]].double()
            means[:, d] = means[:, d].index_add(0, row, v) / count
        uniq = uniq[chosen]
        coords = torch.stack([torch.full_like(uniq, f), uniq // (dims[0] * dims[1]), uniq // dims[0] % dims[1],
                              uniq % dims[0]], 1)
        out.append((coords, count, means, index))
        off.append(off[-1] + V)
        at += n
    return [torch.cat([o[k] for o in out]) for k in range(4)] + [torch.tensor(off, dtype=torch.int64, device=DEV)]


def _selected(c, d, off, ego):
    """The selector's definition, in 64 bits."""
    q = mmbev.DEFAULT_POLICY
    rois, budgets, roi_off, sweeps = [], [], [0], []
    ttc, flags, rank = np.full(len(d), np.inf), np.zeros(len(d), np.int64), np.zeros(len(d), np.int64)
    for f, e in enumerate(ego):
        D = d[off[f]:off[f + 1]]
        cs, sn, v = math.cos(e["dyaw"]), math.sin(e["dyaw"]), float(e["speed"])
        turn = lambda x, y: (cs * x - sn * y, sn * x + cs * y)  # noqa: E731
        old = np.stack(turn(D["x"], D["y"])) + np.array([[e["dx"]], [e["dy"]]])
        new = np.stack(turn(D["x"] + D["vx"] * q["dt"], D["y"] + D["vy"] * q["dt"])) + np.array([[e["dx"]], [e["dy"]]])
        w = np.stack(turn(D["vx"], D["vy"])) - np.array([[v], [0.0]])
        far, reach = np.hypot(*new), max(q["d_min"], v * v / (2 * q["a_brake"]))
        part = min(1.0, max(0.0, (v - q["speed_wide"]) / (q["speed_narrow"] - q["speed_wide"])))
        cone = math.radians(q["theta_max_deg"] + part * (q["theta_min_deg"] - q["theta_max_deg"]))
        geom = (new[0] >= 0) & (far <= reach) & (np.arctan2(np.abs(new[1]), new[0]) <= cone)
        ww = (w * w).sum(0)
        t = -(new * w).sum(0) / np.where(ww > 0, ww, 1.0)
        hit = (ww > 0) & (t > 0) & (np.hypot(*(new + t * w)) <= q["r_coll"])
        t = np.where(hit, t, np.inf)
        safe = (D["cls"] != 2) & (t <= np.where(D["cls"] == 0, q["tau_vru"], q["tau_motorized"]))
        must = geom | safe
        order = np.lexsort((np.arange(len(D)), far, t, ~must))
        n = q["n_reduced"] if v < q["slow_speed"] or len(D) >= q["dense_count"] else q["n_full"]
        ahead = int(must.sum())
        for r, i in enumerate(order):
            dropped = not must[i] and r - ahead >= q["max_optional"]
            yaw = D["yaw"][i] + e["dyaw"]
            ext = [D["length"][i] / 2 + q["margin"], D["width"][i] / 2 + q["margin"]]
            rois += [[*old[:, i], math.cos(yaw), math.sin(yaw), *ext, 0.0, 0.0],
                     [*new[:, i], math.cos(yaw), math.sin(yaw), *ext, 0.0, 0.0]]
            budgets += 2 * [q["n_full"] if must[i] else 0 if dropped else n]
            k = off[f] + i
            rank[k], ttc[k] = r, t[i]
            flags[k] = geom[i] + 2 * safe[i] + 4 * must[i] + 8 * dropped
        roi_off.append(len(rois))
        sweeps.append(n)
    return [np.array(rois), np.array(budgets), np.array(roi_off), ttc, flags, rank, np.array(sweeps)]


def exact(c, seed):
    if c["kind"] == "clusters":
        return None  # whole numbers only
    if c["kind"] == "selector":
        return _selected(c, *_detections(c, seed))
    s = _inputs(c, seed)
    coords, counts, means, index, off = _voxels(s)
    n = len(coords)
    if c["kind"] == "bev":
        full = torch.zeros((c["frames"], c["features"], c["dz"], c["dy"], c["dx"]), dtype=torch.float64, device=DEV)
        b, z, y, x = coords.unbind(1)
        for k in range(c["features"]):
            full[b, k, z, y, x] = means[:, k]
        return full.view(c["frames"], -1, c["dy"], c["dx"])
    rows = c["frames"] * c["max_voxels"]
    out = [torch.full((rows, 4), -7, device=DEV), torch.full((rows,), -7, device=DEV),
           torch.full((rows, c["features"]), -7.0, dtype=torch.float64, device=DEV),
           torch.full((rows, c["max_points"]), -7, device=DEV), off]
    for full, part in zip(out, (coords, counts, means, index)):
        full[:n] = part
    return out

"""Performance cases of the framework's public entry points.

Each case is one pass that a mapping program runs: a frame through
`Context.voxelize` and `Context.fit_predict`, a batch of scans through either,
a captured fit replayed, a stream of frames through a fresh `Map`, the initial
Gaussians of a frame and its structure loss. Sizes and hyper-parameters are
those of the workload presets (`configs.WORKLOADS`), of the serving streams
(`synth.STREAM_SENSORS`) and of the tests (odd grids, caps and voxel sizes).

Inputs are LiDAR scans of the box scene of `synth`, ray-cast here on the GPU
with torch, so that a frame takes milliseconds. A case fixes the scene, the
poses and which voxel every return falls in; the seed moves the returns inside
their voxels (1 cm and up to a tenth of the voxel) and sets where the scan
starts, so that every seed gives outputs of the same shapes. Launch choices
are those a program takes: the autotuner's cached ones where the cache has the
case's (grid, cap, precision), the library's defaults elsewhere. MIXED
precision is left out: on every preset it is slower than both other forms, and
a program has no reason to choose it.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2410_17084_amd import autotune, synth, vgpr

PRECISION = {"fp32": 0, "fp64": 2}


# ---------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------
def _case(name, op, scan="spin", beams=32, azimuths=1800, frames=1, voxel=0.5, cap=128, tau=3, grid=8, ell=0.25,
          ls_mode=0, frame_mode=0, precision="fp32", point_noise=False, n_r=4, cell=0.05):
    c = dict(op=op, scan=scan, beams=beams, azimuths=azimuths, frames=frames, voxel=voxel, cap=cap, tau=tau,
             grid=grid, ell=ell, ls_mode=ls_mode, frame_mode=frame_mode, precision=precision,
             point_noise=point_noise, n_r=n_r, cell=cell)
    if name:
        c["name"] = name
    return c


_PAPER = dict(voxel=0.2, cap=64, tau=10, grid=9, ell=0.1)                       # the paper-shaped stream
_AGGREGATED = dict(scan="aggregated", beams=128, azimuths=1024, frames=10, voxel=0.1, cap=512, tau=3, grid=16,
                   ell=0.05, ls_mode=1)                                        # the large map update


def listed():
    return [
        # a scan of the smallest sensor of the serving streams, one at a time: launches and waits count
        _case("frame_16x512", "frame", beams=16, azimuths=512),
        # one ordinary spinning scan, voxelized and fitted as it arrives
        _case("frame_32x1800", "frame"),
        # the same scan's fit replayed as a captured graph, the latency form of the batched fit
        _case("graph_32x1800", "graph"),
        # a log of 64 scans keyed and sorted in one call (2.4M points): the largest sort
        _case("voxelize_64_scans", "voxelize", frames=64),
        # ... and fitted in one call: many small voxels on a small grid
        _case("fit_64_scans", "fit", frames=64),
        # 16 dense scans, spinning and rosette, at 1 m in FP64: medium and large voxels
        _case("fit_16_scans_fp64", "fit", scan="mixed", beams=128, azimuths=1024, frames=16, voxel=1.0, cap=256,
              ell=0.5, precision="fp64"),
        # the headline: a 1M-point aggregated frame, voxelized and fitted, voxels up to the 512 cap, 16 x 16 grid
        _case("step_aggregated", "frame", **_AGGREGATED),
        # the PCA-rotated frame with a per-point noise variance, odd sizes throughout
        _case("fit_rotated_noise", "fit", beams=64, azimuths=1031, voxel=0.37, cap=201, tau=5, grid=11, ell=0.2,
              ls_mode=1, frame_mode=1, point_noise=True),
        # ten frames of one sensor through a fresh map (voxels re-solved on their stored points)
        _case("map_64x1024", "map", beams=64, azimuths=1024, frames=10, **_PAPER),
        # the same update with the covariance-centred state (81 carried rows a voxel)
        _case("map_feedback_64x1024", "map_feedback", beams=64, azimuths=1024, frames=6, **_PAPER),
        # the initial Gaussians of the aggregated frame's grids
        _case("gauss_aggregated", "gauss", **_AGGREGATED),
        # the structure loss of the aggregated frame against its 2.6M Gaussian rows
        _case("loss_aggregated", "loss", **_AGGREGATED),
    ]


def draw(rng):
    op = rng.choice(["frame", "frame", "fit", "fit", "voxelize", "graph", "map", "map_feedback", "gauss", "loss"])
    beams = rng.choice([16, 20, 32, 40, 64, 100, 128])
    az = int(round(math.exp(rng.uniform(math.log(300), math.log(2048)))))
    most = {"voxelize": 64, "map": 10, "map_feedback": 6}.get(op, 8)
    top = 2_000_000 if op == "voxelize" else 400_000
    frames = int(round(math.exp(rng.uniform(0.0, math.log(most)))))
    frames = max(1, min(frames, top // (beams * az)))
    low = 0.1 if frames * beams * az > 150_000 else 0.25  # a thin scan fills no small voxels
    voxel = round(math.exp(rng.uniform(math.log(low), math.log(1.0))), 3)
    grid = rng.randint(4, 16)
    n_r = rng.choice([d for d in (1, 2, 3, 4, 5) if grid % d == 0])
    cap = int(round(math.exp(rng.uniform(math.log(24), math.log(512)))))
    tau = rng.choice([3, 3, 3, 5, 10])
    if op in ("map", "map_feedback"):  # a frame's voxels hold a scan's few points: they must reach tau to be solved
        grid, cap, tau, voxel = min(grid, 12), min(cap, 128), min(tau, 5), max(voxel, 0.25)
    scan = "spin"
    if op in ("frame", "fit", "voxelize") and rng.random() < 0.3:
        scan = rng.choice(["mixed", "aggregated"])
    return _case(None, op, scan=scan, beams=beams, azimuths=az, frames=frames, voxel=voxel, cap=cap,
                 tau=tau, grid=grid, ell=round(voxel * rng.uniform(0.3, 0.7), 4),
                 ls_mode=rng.choice([0, 0, 1]), frame_mode=rng.choice([0, 0, 0, 1]) if op in ("frame", "fit") else 0,
                 precision=rng.choice(["fp32", "fp32", "fp64"]), point_noise=op == "fit" and rng.random() < 0.3,
                 n_r=n_r, cell=round(max(0.03, voxel * n_r / grid * rng.uniform(1.0, 3.0)), 3))


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _cast(boxes, origin, dirs, gen):
    """Points of rays (origin (F, 1, 3), dirs (F, R, 3)) against the ground and the boxes, 2 cm range noise."""
    far = torch.full(dirs.shape[:2], math.inf, device="cuda")
    t = torch.where(dirs[..., 2] < -1e-9, -origin[..., 2] / dirs[..., 2], far)
    inv = 1.0 / dirs
    for lo, hi in zip(boxes.lo.tolist(), boxes.hi.tolist()):
        a = (torch.tensor(lo, device="cuda") - origin) * inv
        b = (torch.tensor(hi, device="cuda") - origin) * inv
        near, away = torch.minimum(a, b).amax(-1), torch.maximum(a, b).amin(-1)
        t = torch.where((away >= near) & (near > 1e-6), torch.minimum(t, near), t)
    hit = t <= 120.0
    t = t + 0.02 * torch.randn(t.shape, device="cuda", generator=gen)
    return [(origin[f] + t[f, :, None] * dirs[f])[hit[f]].contiguous() for f in range(len(dirs))]


def _spin(c, boxes, positions, yaws, gen):
    d = torch.from_numpy(synth.spin_directions(c["beams"], c["azimuths"])).float().cuda()
    return _turned(d, boxes, positions, yaws, gen)


def _turned(d, boxes, positions, yaws, gen):
    out = []
    for f in range(0, len(positions), 16):  # 16 scans at a time
        yaw = torch.tensor(yaws[f:f + 16], device="cuda")[:, None]
        cs, sn = torch.cos(yaw), torch.sin(yaw)
        dd = torch.stack([cs * d[:, 0] - sn * d[:, 1], sn * d[:, 0] + cs * d[:, 1], d[:, 2].expand(len(yaw), -1)], -1)
        out += _cast(boxes, torch.tensor(positions[f:f + 16], device="cuda")[:, None, :], dd, gen)
    return out


def _gen(seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    return gen


def _frames(c, seed):
    """The case's scans as a list of (n, 3) float32 GPU tensors: the returns of `_scans`, moved inside their
    voxels (folded back at the faces) and rolled to another first return."""
    gen, s = _gen(seed), float(np.float32(c["voxel"]))
    out = []
    for p in _scans(c):
        k = torch.floor(p.double() * (1.0 / s))
        f = p.double() / s - k
        f = f + min(0.01 / s, 0.1) * torch.randn(f.shape, dtype=torch.float64, device="cuda", generator=gen)
        f = (1.0 - (1.0 - f.abs()).abs()).clamp(2e-3, 1.0 - 2e-3)
        start = int(torch.randint(len(p), (1,), device="cuda", generator=gen))
        out.append(((k + f) * s).float().roll(start, 0).contiguous())
    return out


def _scans(c):
    r = np.random.Generator(np.random.PCG64(2410))
    gen = _gen(17084)
    k = c["frames"]
    if c["op"] in ("map", "map_feedback"):  # one sensor driving through a clearing, about 3 m/s at 10 Hz
        step, head, yaw0 = r.uniform(0.2, 0.4), r.uniform(0, 2 * np.pi), r.uniform(0, 2 * np.pi)
        pos = [[i * step * math.cos(head), i * step * math.sin(head), 1.8] for i in range(k)]
        return _spin(c, synth.box_scene(clear_radius=12.0), pos, [yaw0 + 0.02 * i for i in range(k)], gen)
    if c["scan"] == "aggregated":  # scans 0.05 m apart with 1 cm registration noise, near surfaces kept
        head, at = r.uniform(0, 2 * np.pi), r.uniform(-1, 1, 2)
        pos = [[at[0] + 0.05 * i * math.cos(head), at[1] + 0.05 * i * math.sin(head), 1.8] for i in range(k)]
        pos = (np.array(pos) + r.normal(0, 0.01, (k, 3))).tolist()
        return _spin(c, synth.box_scene(clear_radius=2.0), pos, [head] * k, gen)
    rad, phi, yaw = 2 * np.sqrt(r.uniform(size=k)), r.uniform(0, 2 * np.pi, k), r.uniform(0, 2 * np.pi, k).tolist()
    pos = np.stack([rad * np.cos(phi), rad * np.sin(phi), np.full(k, 1.8)], 1).tolist()
    boxes = synth.box_scene()
    if c["scan"] != "mixed":
        return _spin(c, boxes, pos, yaw, gen)
    rays = min(100_000, c["beams"] * c["azimuths"])  # every second scan is a rosette, pitched down by 10 degrees
    p = math.radians(-10.0)
    pitch = np.array([[math.cos(p), 0, -math.sin(p)], [0, 1, 0], [math.sin(p), 0, math.cos(p)]])
    d = torch.from_numpy(synth.rosette_directions(rays, 0.0) @ pitch.T).float().cuda()
    spins, petals = _spin(c, boxes, pos[0::2], yaw[0::2], gen), _turned(d, boxes, pos[1::2], yaw[1::2], gen)
    return [(petals if i % 2 else spins)[i // 2] for i in range(k)]


def _cloud(c, seed):
    """The case's points and frame offsets (an aggregated frame is one frame)."""
    f = _frames(c, seed)
    if c["scan"] == "aggregated":
        f = [torch.cat(f)]
    return torch.cat(f), [0] + np.cumsum([len(x) for x in f]).tolist()


def _params(c):
    return vgpr.default_params(voxel_size=c["voxel"], max_pts=c["cap"], min_pts=c["tau"], grid_side=c["grid"],
                               signal_var=1.0, length_scale=c["ell"], noise_var=1e-3, ls_mode=c["ls_mode"],
                               frame_mode=c["frame_mode"], precision=PRECISION[c["precision"]], converge_var=0.3)


def _point_noise(c, n, seed):
    """Per-point sensor variances between 2 and 6 cm^2 (range-dependent in a real sensor)."""
    if not c["point_noise"]:
        return None
    gen = _gen(seed + 77)
    return 2e-4 + 4e-4 * torch.rand(n, device="cuda", generator=gen)


def _grids(c, seed):
    """Predicted grids as a fit of the frame leaves them, made with torch: per voxel a tilted patch on its
    face with variances between 1e-4 and 1e-1, NaN rows for voxels below tau; (rows, status)."""
    xyz, _ = _cloud(c, seed)
    g = _group(xyz, c["voxel"])
    V, m, s = len(g["cnt"]), c["grid"] ** 2, c["voxel"]
    gen = _gen(seed + 5)
    sums = torch.zeros((V, 6), dtype=torch.float64, device="cuda")
    p = xyz.double()
    sums.index_add_(0, g["vox"], torch.cat([p, p * p], 1))
    mean = sums[:, :3] / g["cnt"][:, None]
    ax = (sums[:, 3:] / g["cnt"][:, None] - mean * mean).argmin(1)
    q = (torch.arange(c["grid"], device="cuda", dtype=torch.float64) + 0.5) / c["grid"]
    i, j = (t.reshape(1, m) for t in torch.meshgrid(q, q, indexing="ij"))
    k = g["idx"].double()
    rows = torch.empty((V, m, 4), dtype=torch.float32, device="cuda")
    tilt = 0.3 * torch.randn((V, 2), device="cuda", generator=gen, dtype=torch.float64)
    for a in range(3):
        v = torch.nonzero(ax == a)[:, 0]
        for b, t in (((a + 1) % 3, i), ((a + 2) % 3, j)):
            rows[v, :, b] = ((k[v, b, None] + t) * s).float()
        rows[v, :, a] = (mean[v, a, None] + s * (tilt[v, :1] * (i - 0.5) + tilt[v, 1:] * (j - 0.5))).float()
    rows[..., :3] += 0.005 * s * torch.randn((V, m, 3), device="cuda", generator=gen)
    rows[..., 3] = torch.exp(torch.empty((V, m), device="cuda").uniform_(math.log(1e-4), math.log(1e-1),
                                                                           generator=gen))
    solved = g["cnt"] >= c["tau"]
    rows[~solved] = math.nan
    return rows, torch.where(solved, 1, 2).to(torch.uint8)


def _gaussians(c, seed):
    """Gaussians as `gauss_init` leaves them for such grids (position, weight, variances, 0): the mean and the
    scatter of every n_r x n_r subgrid."""
    rows, status = _grids(c, seed)
    V, gs, nr = len(rows), c["grid"], c["n_r"]
    ns = gs // nr
    r = rows.reshape(V, ns, nr, ns, nr, 4).transpose(2, 3).reshape(V, ns * ns, nr * nr, 4)
    out = torch.zeros((V, ns * ns, 8), device="cuda")
    out[..., :3] = r[..., :3].mean(2)
    out[..., 3] = (1.0 / r[..., 3]).sum(2)
    out[..., 4:7] = r[..., :3].var(2, unbiased=False) if nr > 1 else 0.0 * r[:, :, 0, :3]
    return out


def _context(c, p, stream=None):
    ctx = vgpr.Context(0, stream=stream)
    d = torch.cuda.get_device_properties(0)
    tuned = autotune.load_cached(p, f"{d.gcnArchName.split(':')[0]}x{d.multi_processor_count}cu")
    if tuned is not None and c["op"] in ("frame", "fit", "graph"):
        ctx.set_tuning(vgpr.Tuning.from_dict(tuned["tuning"]))
    return ctx


def _update_buffers(c, frames):
    """The output buffers that a program keeps for a map's updates, one set a frame, as many rows as the frame
    touches voxels with enough points."""
    bufs, seen = [], None
    for f in frames:
        seen = f if seen is None else torch.cat([seen, f])
        cap = int(_due(c, seen, f)[1].sum())
        bufs.append((torch.zeros(cap, dtype=torch.int64, device="cuda"),
                     torch.zeros((cap, c["grid"] ** 2, 4), device="cuda"),
                     torch.zeros(cap, dtype=torch.int8, device="cuda"),
                     torch.zeros(cap, dtype=torch.uint8, device="cuda")))
    return bufs


def _due(c, seen, frame):
    """Voxels of all points so far, and which of them this frame touched with at least tau points held."""
    g, now = _group(seen, c["voxel"]), _group(frame, c["voxel"])["key"]
    return g, torch.isin(g["key"], now) & (g["cnt"].clamp(max=c["cap"]) >= c["tau"])


def prepare(case, seed):
    c, op = case, case["op"]
    p = _params(c)
    s = dict(op=op, c=c, p=p)
    if op in ("map", "map_feedback"):
        s["frames"] = _frames(c, seed)
        s["out"] = _update_buffers(c, s["frames"])
        s["max_voxels"] = len(_group(torch.cat(s["frames"]), c["voxel"])["cnt"]) * 5 // 4
        s["ctx"] = _context(c, p)
        return s
    if op == "gauss":
        s["rows"], s["status"] = _grids(c, seed)
        s["ctx"] = _context(c, p)
        return s
    s["xyz"], s["offsets"] = _cloud(c, seed)
    if op == "loss":
        s["gauss"] = _gaussians(c, seed)
        s["ctx"] = _context(c, p)
        return s
    if op == "graph":  # capture needs a stream of its own; the frame's voxels are in hand
        s["stream"] = torch.cuda.Stream()
        s["stream"].wait_stream(torch.cuda.current_stream())
        s["ctx"] = _context(c, p, s["stream"])
        with torch.cuda.stream(s["stream"]):
            s["vox"] = s["ctx"].voxelize(s["xyz"], p, s["offsets"])
            s["graph"] = s["ctx"].fit_graph(s["xyz"], s["vox"], p)
        return s
    s["ctx"] = _context(c, p)
    s["noise"] = _point_noise(c, len(s["xyz"]), seed)
    if op == "fit":
        s["vox"] = s["ctx"].voxelize(s["xyz"], p, s["offsets"])
    return s


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------
def run(s):
    op, ctx, p, c = s["op"], s["ctx"], s["p"], s["c"]
    if op in ("map", "map_feedback"):
        m = vgpr.Map(ctx, p, max_voxels=s["max_voxels"], feedback=op == "map_feedback")
        n_upd = []
        for f, out in zip(s["frames"], s["out"]):
            n_upd.append(len(m.update(f, cap_upd=len(out[0]), out=out)[0]))
        m.close()
        return [dict(n_upd=n, keys=k, out=o, axis=a, status=t) for n, (k, o, a, t) in zip(n_upd, s["out"])]
    if op == "gauss":
        return ctx.gauss_init(s["rows"], s["status"], c["grid"], c["n_r"])
    if op == "loss":
        loss, n, value, arg = ctx.structure_loss(s["xyz"], s["gauss"], c["cell"], 1)
        return dict(loss=loss, n=n, value=value, arg=arg)
    if op == "graph":
        out, axis, status = s["graph"].launch()
        return dict(out=out, axis=axis, status=status)
    if op == "fit":
        out, axis, status = ctx.fit_predict(s["xyz"], s["vox"], p, noise_var=s["noise"])
        return dict(out=out, axis=axis, status=status)
    v = ctx.voxelize(s["xyz"], p, s["offsets"])
    got = dict(keys=v.keys, offsets=v.offsets, counts=v.counts, perm=v.perm,
               frame_vox=np.array(v.frame_vox))
    if op == "frame":
        out, axis, status = ctx.fit_predict(s["xyz"], v, p, noise_var=s["noise"])
        got.update(out=out, axis=axis, status=status)
    return got


# ---------------------------------------------------------------------------
# the work of a pass and its values in 64 bits, in plain torch
# ---------------------------------------------------------------------------
def _group(xyz, voxel, offsets=None):
    """Voxels by (frame, key): sorted point order, voxel of each point, and per voxel count, start, indices."""
    k = torch.floor(xyz.double() * (1.0 / float(np.float32(voxel)))).long()
    key = ((k[:, 0] + (1 << 20)) << 42) | ((k[:, 1] + (1 << 20)) << 21) | (k[:, 2] + (1 << 20))
    order = torch.sort(key, stable=True)[1]
    if offsets is not None and len(offsets) > 2:
        cuts = torch.tensor(offsets[1:-1], device="cuda")
        fr = torch.bucketize(torch.arange(len(xyz), device="cuda"), cuts, right=True)
        order = order[torch.sort(fr[order], stable=True)[1]]
        both = torch.stack([fr[order], key[order]], 1)
    else:
        both = key[order, None]
    head = torch.ones(len(xyz), dtype=torch.bool, device="cuda")
    head[1:] = (both[1:] != both[:-1]).any(1)
    rank = torch.cumsum(head, 0) - 1
    vox = torch.empty_like(rank)
    vox[order] = rank
    start = torch.nonzero(head)[:, 0]
    cnt = torch.diff(start, append=torch.tensor([len(xyz)], device="cuda"))
    return dict(order=order, vox=vox, start=start, cnt=cnt, idx=k[order[start]], key=key[order[start]])


def _solve_flops(n, m):
    n = n.double()
    return float((n ** 3 / 3 + n * n * m + 2 * n * n + 4 * n * m + 6 * (n * n / 2 + n * m)).sum())


def work(case):
    c, op, m = case, case["op"], case["grid"] ** 2
    if op in ("map", "map_feedback"):
        by, fl, seen = 0.0, 0.0, None
        for f in _frames(c, 0):
            seen = f if seen is None else torch.cat([seen, f])
            g, due = _due(c, seen, f)
            n = g["cnt"].clamp(max=c["cap"])[due]  # each touched voxel solved once a frame at most
            by += 12.0 * len(f) + float((12.0 * n).sum()) + len(n) * (16.0 * m + 10)
            fl += _solve_flops(n, m)
        return dict(bytes=by, flops=fl)
    xyz, offsets = _cloud(c, 0)
    g = _group(xyz, c["voxel"], offsets)
    V, n = len(g["cnt"]), g["cnt"].clamp(max=c["cap"])
    n = n[n >= c["tau"]]
    ns = c["grid"] // c["n_r"]
    if op == "gauss":  # rows of the solved voxels, a status byte of each, 32 bytes a Gaussian
        return dict(bytes=16.0 * m * len(n) + V + 32.0 * V * ns * ns, flops=30.0 * m * len(n))
    if op == "loss":  # the points, the Gaussians, value and index a point; one distance a point at the least
        return dict(bytes=(12.0 + 8.0) * len(xyz) + 32.0 * V * ns * ns, flops=10.0 * len(xyz))
    by, fl = 0.0, 0.0
    if op in ("voxelize", "frame"):
        by, fl = by + 16.0 * len(xyz) + 16.0 * V, fl + 3.0 * len(xyz)
    if op != "voxelize":
        by, fl = by + float((12.0 * n).sum()) + V * (16.0 * m + 18), fl + _solve_flops(n, m)
    return dict(bytes=by, flops=fl)


def _posterior(P, n, idx, noise, c):
    """Posterior rows (V, m, 4) in float64 of voxels with points P (V, N, 3), n of them kept, voxel indices idx
    and noise variances (V, N), by the Cholesky factor of K + S."""
    V, N = P.shape[:2]
    s, nq = float(np.float32(c["voxel"])), c["grid"]
    dev = dict(dtype=torch.float64, device="cuda")
    mask = torch.arange(N, device="cuda") < n[:, None]
    mean = (P * mask[..., None]).sum(1) / n[:, None]
    D = (P - mean[:, None]) * mask[..., None]
    C = torch.stack([(D * D[..., a:a + 1]).sum(1) for a in range(3)], 1) / n[:, None, None]
    w, U = np.linalg.eigh(C.cpu().numpy())
    w, v = torch.from_numpy(w).cuda(), torch.from_numpy(np.ascontiguousarray(U[:, :, 0])).cuda()
    ax = v.abs().argmax(1)
    ell = torch.full((V,), float(np.float32(c["ell"])), **dev)
    if c["ls_mode"] == 1:
        ell = (math.sqrt(3.0) * ((w[:, 1] + w[:, 2]) * 0.5).clamp(min=0).sqrt()).clamp(0.05 * s, 2.0 * s)
    lam = (1.0 / (2.0 * ell * ell))[:, None, None]
    t = (torch.arange(nq, **dev) + 0.5) / nq
    ti, tj = (x.reshape(1, -1) for x in torch.meshgrid(t, t, indexing="ij"))

    def at(A, i):
        return torch.gather(A, -1, i.view(-1, *[1] * (A.dim() - 1)).expand(*A.shape[:-1], 1))[..., 0]

    if c["frame_mode"] == 1:
        v = v * torch.where(at(v, ax) < 0, -1.0, 1.0)[:, None]
        e = torch.eye(3, **dev)[v.abs().argmin(1)]
        e1 = torch.linalg.cross(e, v)
        e1 = e1 / e1.norm(dim=1, keepdim=True)
        e2 = torch.linalg.cross(v, e1)
        xu, xw, f = ((D * b[:, None]).sum(-1) for b in (e1, e2, v))
        gu, gw = (((x - 0.5) * s).float().double().expand(V, -1) for x in (ti, tj))
        qu, qw = gu, gw
    else:
        u, o = (ax + 1) % 3, (ax + 2) % 3
        ku, kw = (at(idx, a).double()[:, None] for a in (u, o))
        xu, xw, f = at(P, u) - ku * s, at(P, o) - kw * s, at(D, ax)
        gu, gw = ((k + x).mul(s).float().double() for k, x in ((ku, ti), (kw, tj)))
        qu, qw = gu - ku * s, gw - kw * s
    both = mask[:, :, None] & mask[:, None, :]
    K = torch.exp(-((xu[:, :, None] - xu[:, None]) ** 2 + (xw[:, :, None] - xw[:, None]) ** 2) * lam) * both
    K = K + torch.diag_embed(torch.where(mask, noise, 1.0))
    Q = torch.exp(-((xu[:, :, None] - qu[:, None]) ** 2 + (xw[:, :, None] - qw[:, None]) ** 2) * lam) * mask[..., None]
    L = torch.linalg.cholesky(K)
    Z = torch.cat([Q, (f * mask)[..., None]], -1)
    for j in range(N):  # forward substitution
        if j:
            Z[:, j:j + 1] -= torch.bmm(L[:, j:j + 1, :j].contiguous(), Z[:, :j])
        Z[:, j] /= L[:, j, j, None]
    y, Z = Z[..., -1:], Z[..., :-1]
    var, fq = (1.0 - (Z * Z).sum(1)).clamp(min=0), (Z * y).sum(1)
    rows = torch.empty((V, nq * nq, 4), **dev)
    rows[..., 3] = var
    if c["frame_mode"] == 1:
        for a in range(3):
            rows[..., a] = mean[:, a, None] + gu * e1[:, a, None] + gw * e2[:, a, None] + fq * v[:, a, None]
        return rows
    for a in range(3):
        k = ax == a
        rows[k, :, a] = mean[k, a, None] + fq[k]
        rows[k, :, (a + 1) % 3], rows[k, :, (a + 2) % 3] = gu[k], gw[k]
    return rows


def _solve_all(P, noise, start, n, idx, c, tau):
    """Rows of every voxel whose n points are P[start:start + n] (NaN below tau), in batches of similar size."""
    m = c["grid"] ** 2
    out = torch.full((len(n), m, 4), math.nan, dtype=torch.float64, device="cuda")
    at = torch.nonzero(n >= tau)[:, 0]
    at = at[torch.sort(n[at])[1]]
    sizes, a = n[at].tolist(), 0
    while a < len(at):
        b, N = a, sizes[a]
        while b < len(at) and sizes[b] <= max(8, 1.25 * sizes[a]) and (b - a) * sizes[b] * (sizes[b] + m) < 1 << 27:
            N = sizes[b]
            b += 1
        v = at[a:b]
        i = (start[v, None] + torch.arange(N, device="cuda")).clamp(max=len(P) - 1)
        out[v] = _posterior(P[i], n[v], idx[v], noise[i], c)
        a = b
    return out


def _exact_map(c, seed):
    """The stored-point map: every touched voxel solved on the first `cap` of all points that reached it, until
    its largest variance is at most 0.3."""
    seen, done, got = None, torch.empty(0, dtype=torch.long, device="cuda"), []
    for f in _frames(c, seed):
        seen = f if seen is None else torch.cat([seen, f])
        g, due = _due(c, seen, f)
        n, v = g["cnt"].clamp(max=c["cap"]), due & ~torch.isin(g["key"], done)
        P = seen[g["order"]].double()
        rows = _solve_all(P, torch.full((len(P),), float(np.float32(1e-3)), dtype=torch.float64, device="cuda"),
                          g["start"][v], n[v], g["idx"][v], c, c["tau"])
        done = torch.cat([done, g["key"][v][rows[..., 3].amax(1) <= float(np.float32(0.3))]])
        whole = torch.zeros((int(due.sum()), c["grid"] ** 2, 4), dtype=torch.float64, device="cuda")
        whole[:len(rows)] = rows
        got.append(dict(n_upd=None, keys=None, out=whole, axis=None, status=None))
    return got


def exact(case, seed):
    c, op = case, case["op"]
    if op in ("voxelize", "map_feedback"):  # whole numbers; rows carried on as float32 from solve to solve
        return None
    if op == "map":
        return _exact_map(c, seed)
    if op == "gauss":
        rows, status = _grids(c, seed)
        V, gs, nr = len(rows), c["grid"], c["n_r"]
        ns = gs // nr
        r = rows.double().reshape(V, ns, nr, ns, nr, 4).transpose(2, 3).reshape(V, ns * ns, nr * nr, 4)
        w = 1.0 / r[..., 3:].clamp(min=float(np.float32(1e-8)))
        sw = w.sum(2)
        mean = (w * r[..., :3]).sum(2) / sw
        S = (w * (r[..., :3] - mean[:, :, None]) ** 2).sum(2) / sw
        out = torch.cat([mean, sw, S, torch.zeros_like(sw)], -1)
        out[status != 1] = math.nan
        return out
    xyz, offsets = _cloud(c, seed)
    if op == "loss":
        G = _gaussians(c, seed).reshape(-1, 8)
        G = G[torch.isfinite(G).all(1)].double()
        if len(xyz) * len(G) > 4e10:
            return None
        S = G[:, 4:7].sqrt().mean(1)
        value = torch.cat([(sum((p[:, a, None] - G[:, a]) ** 2 for a in range(3)).sqrt() - S).amin(1)
                           for p in xyz.double().split(max(1, (1 << 26) // max(1, len(G))))])
        return dict(loss=float(value.mean()), n=None, value=value, arg=None)
    g = _group(xyz, c["voxel"], offsets)
    noise = _point_noise(c, len(xyz), seed)
    noise = torch.full((len(xyz),), 1e-3, device="cuda") if noise is None else noise[g["order"]]
    rows = _solve_all(xyz[g["order"]].double(), noise.double(), g["start"], g["cnt"].clamp(max=c["cap"]), g["idx"], c,
                      c["tau"])
    got = dict(out=rows, axis=None, status=None)
    if op == "frame":
        got.update(keys=None, offsets=None, counts=None, perm=None, frame_vox=None)
    return got

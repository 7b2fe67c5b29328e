"""Performance cases of the framework: the calls its users make, through the
public Python entry points, over the sizes they are made with.

Kinds (the "kind" of a case):
  depth    one mapping session: clear a volume, integrate a run of depth maps
           taken along a street, read the map back
  laser    the same with the returns of a spinning laser scanner
  reg      one regularisation of a fused map (and its state read back): FP32
           or 16-bit state, quadratic or L1 data term, fixed or accelerated
           steps, with or without stopping at a gap
  batch    many uneven sub-maps regularised in one call
  surface  the zero-crossing points, the mesh and its area of a map
  warm     the learned warm start of a whole map
  train    one training step of the network (loss gradient and Adam)
  forward  the network on given tiles

Inputs come from a procedural street (road, facades with a seeded set-back
per 10 m, parked cars, an end wall): depth maps and laser scans ray-cast
against its boxes, and fused fields evaluated from its signed distance with
noise, observed in front of the surfaces and to mu behind them.
"""
import math

import numpy as np
import torch

from paper_1604_03734_amd import denser as D
from paper_1604_03734_amd import warmstart

LAM = 0.5
STEP = 1.0 / math.sqrt(12.0)
STORAGE = {"f32": D.DN_F32, "f16": D.DN_F16, "bf16": D.DN_BF16}
STREET_LEN = 100.0            # metres of street before a map goes on with another copy beside it
COPY_PITCH = 24               # blocks between copies
ROOM = 4096                   # blocks of the arrays a mapping session keeps its map in
VOX = 0.2                     # metres, the street workload's voxel edge
MU = 0.6
F64 = torch.float64


def listed():
    return [
        # a small indoor-size session at fine voxels: launches and host work decide
        {"name": "depth_small", "kind": "depth", "width": 320, "height": 96, "frames": 4,
         "voxel": 0.1, "max_depth": 20.0},
        # a car driving down a street, full-size stereo depth maps
        {"name": "depth_street", "kind": "depth", "width": 1242, "height": 375, "frames": 12,
         "voxel": 0.2, "max_depth": 50.0},
        # a spinning scanner on the same street, every few metres
        {"name": "laser_street", "kind": "laser", "rings": 64, "azimuths": 1024, "scans": 3,
         "voxel": 0.2, "max_depth": 50.0},
        # a small map regularised for a fixed number of iterations
        {"name": "reg_small", "kind": "reg", "blocks": 503, "iters": 200, "storage": "f32",
         "data": "l2", "gamma": 0.0, "gap_every": 0},
        # one street solved to a relative gap of 1e-3 with the accelerated steps
        {"name": "reg_street_gap", "kind": "reg", "blocks": 5777, "iters": 400, "storage": "f32",
         "data": "l2", "gamma": 0.5, "gap_every": 10},
        # a district: the map is far larger than the caches
        {"name": "reg_district", "kind": "reg", "blocks": 202195, "iters": 30, "storage": "f32",
         "data": "l2", "gamma": 0.0, "gap_every": 0},
        # the 16-bit state that halves the solver's traffic
        {"name": "reg_bf16", "kind": "reg", "blocks": 60001, "iters": 50, "storage": "bf16",
         "data": "l2", "gamma": 0.0, "gap_every": 0},
        # uneven sub-maps of a city regularised together
        {"name": "batch_submaps", "kind": "batch", "volumes": 16, "lo": 300, "hi": 10000,
         "iters": 60, "data": "l2", "gamma": 0.0},
        # the surface model of one street: points, mesh and area
        {"name": "surface_street", "kind": "surface", "blocks": 5777},
        # warm start of one street before it is solved
        {"name": "warm_street", "kind": "warm", "blocks": 5777},
        # a training step at the trainer's batch size
        {"name": "train_256", "kind": "train", "tiles": 256, "loss_kind": 1},
        # the network on a serving batch
        {"name": "forward_32", "kind": "forward", "tiles": 32},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["depth", "depth", "laser", "reg", "reg", "reg", "reg", "batch", "surface", "warm", "train",
                       "forward"])
    if kind == "depth":
        h = _log_int(rng, 24, 375)
        voxel, far = rng.choice([(0.1, 20.0), (0.2, 50.0), (0.4, 50.0)])
        return {"kind": kind, "width": int(h * 3.3) + rng.randrange(7), "height": h, "frames": rng.randint(1, 12),
                "voxel": voxel, "max_depth": far}
    if kind == "laser":
        voxel, far = rng.choice([(0.1, 20.0), (0.2, 50.0)])
        return {"kind": kind, "rings": rng.randint(4, 64), "azimuths": _log_int(rng, 90, 1024),
                "scans": rng.randint(1, 3), "voxel": voxel, "max_depth": far}
    if kind == "reg":
        blocks = _log_int(rng, 60, 202195)
        iters = max(10, min(500, 6000000 // blocks, rng.randint(20, 500)))
        storage = rng.choice(["f32", "f32", "f16", "bf16"])
        data = rng.choice(["l2", "l2", "l2", "l1"])
        gamma = 0.5 if data == "l2" and rng.random() < 0.4 else 0.0
        return {"kind": kind, "blocks": blocks, "iters": iters, "storage": storage, "data": data, "gamma": gamma,
                "gap_every": rng.choice([0, 0, 10])}
    if kind == "batch":
        lo = _log_int(rng, 50, 1000)
        n = rng.randint(2, 24)
        hi = _log_int(rng, lo + 10, 10000)
        return {"kind": kind, "volumes": n, "lo": lo, "hi": hi, "iters": rng.randint(10, 60),
                "data": rng.choice(["l2", "l2", "l1"]), "gamma": 0.0}
    if kind == "surface":
        return {"kind": kind, "blocks": _log_int(rng, 60, 60000)}
    if kind == "warm":
        return {"kind": kind, "blocks": _log_int(rng, 60, 30000)}
    if kind == "train":
        return {"kind": kind, "tiles": _log_int(rng, 1, 1100), "loss_kind": rng.choice([0, 1])}
    return {"kind": kind, "tiles": _log_int(rng, 1, 1100)}


# ------------------------------------------------------------------ the street
def _dev():
    return torch.device("cuda", torch.cuda.current_device())


def _boxes(seed):
    """Solid boxes [n][2][3] (lo, hi), metres; y points down."""
    rng = np.random.default_rng([seed, 17])
    b = [((-25.0, 1.65, -10.0), (25.0, 4.65, STREET_LEN + 15.0))]
    for j in range(int(STREET_LEN / 10) + 2):
        z0, z1 = 10.0 * j - 5.0, 10.0 * j + 5.0
        for side in (-1.0, 1.0):
            x, h = 7.0 + rng.uniform(0.0, 1.5), rng.uniform(8.0, 16.0)
            lo, hi = (x, x + 3.0) if side > 0 else (-x - 3.0, -x)
            b.append(((lo, -h, z0 - 0.8), (hi, 3.0, z1 + 0.8)))       # solids overlap: no seams inside
    for side in (-1.0, 1.0):
        z = -3.0 + rng.uniform(0.0, 4.0)
        while z < STREET_LEN + 5.0:
            b.append(((side * 5.5 - 0.9, 0.15, z), (side * 5.5 + 0.9, 3.0, z + 4.2)))
            z += 4.2 + rng.uniform(1.0, 6.0)
    b.append(((-20.0, -20.0, STREET_LEN + 10.0), (20.0, 3.0, STREET_LEN + 12.0)))
    return torch.tensor(b, dtype=F64, device=_dev())


def _gen(seed, salt):
    return torch.Generator(device=_dev()).manual_seed(int(seed) * 1009 + salt)


def _cast(boxes, origin, d):
    """Nearest hit parameter of rays origin + t d (float64 [n][3])."""
    best = torch.full((d.shape[0],), math.inf, dtype=F64, device=d.device)
    inv = 1.0 / torch.where(d.abs() < 1e-12, torch.full_like(d, 1e-12), d)
    for lo, hi in boxes:
        t0, t1 = (lo - origin) * inv, (hi - origin) * inv
        tn, tf = torch.minimum(t0, t1).amax(1), torch.maximum(t0, t1).amin(1)
        best = torch.where((tn <= tf) & (tn > 1e-6) & (tn < best), tn, best)
    return best


def _pose(k):
    """Sensor -> world: along the street, weaving a little."""
    yaw = 0.06 * math.sin(0.7 * k)
    T = np.eye(4)
    T[0, 0] = T[2, 2] = math.cos(yaw)
    T[0, 2], T[2, 0] = math.sin(yaw), -math.sin(yaw)
    T[:3, 3] = (0.1 * math.sin(0.3 * k), 0.0, 1.0 * k)
    return T


def _camera(case):
    w, h = case["width"], case["height"]
    f = 700.0 * w / 1242.0
    return (f, f, 0.5 * (w - 1), 0.5 * (h - 1), w, h)


def _depth_maps(case, seed):
    """Stereo depth maps: Gaussian noise in disparity, 5 % invalid pixels."""
    fx, fy, cx, cy, w, h = _camera(case)
    boxes, g, dev = _boxes(seed), _gen(seed, 1), _dev()
    x = (torch.arange(w, dtype=F64, device=dev) - cx) / fx
    y = (torch.arange(h, dtype=F64, device=dev) - cy) / fy
    r = torch.stack([x.expand(h, w), y[:, None].expand(h, w), torch.ones((h, w), dtype=F64, device=dev)], -1)
    maps = []
    for k in range(case["frames"]):
        T = torch.from_numpy(_pose(k)).to(dev)
        z = _cast(boxes, T[:3, 3], r.reshape(-1, 3) @ T[:3, :3].T).reshape(h, w)
        disparity = fx * 0.54 / z + 0.4 * fx / 700.0 * torch.randn((h, w), generator=g, device=dev, dtype=F64)
        z = fx * 0.54 / disparity
        ok = (disparity > 0) & (z <= case["max_depth"]) & (torch.rand((h, w), generator=g, device=dev) >= 0.05)
        maps.append(torch.where(ok, z, torch.zeros_like(z)).float().contiguous())
    return maps


def _scans(case, seed):
    """Returns of a spinning scanner in its own frame; NaN where nothing is hit."""
    boxes, g, dev = _boxes(seed), _gen(seed, 2), _dev()
    el = torch.deg2rad(torch.linspace(-15.0, 15.0, case["rings"], dtype=F64, device=dev))
    az = torch.arange(case["azimuths"], dtype=F64, device=dev) * (2 * math.pi / case["azimuths"])
    e, a = el.repeat_interleave(len(az)), az.repeat(len(el))
    d = torch.stack([torch.cos(e) * torch.sin(a), -torch.sin(e), torch.cos(e) * torch.cos(a)], -1)
    out = []
    for k in range(case["scans"]):
        T = torch.from_numpy(_pose(5 * k)).to(dev)
        r = _cast(boxes, T[:3, 3], d @ T[:3, :3].T)
        r = r + 0.01 * torch.randn(r.shape, generator=g, device=dev, dtype=F64)
        r = torch.where(r <= case["max_depth"], r, torch.full_like(r, math.nan))
        out.append((d * r[:, None]).float().contiguous())
    return out


def _distance(boxes, p):
    """Signed distance (float32 [...]) of points [..., 3] to the union of the boxes."""
    best = torch.full(p.shape[:-1], 1e9, device=p.device)
    for lo, hi in boxes.float():
        q = torch.maximum(lo - p, p - hi)
        m = q.amax(-1)
        best = torch.minimum(best, torch.where(m > 0, q.clamp_min(0).square().sum(-1).sqrt(), m))
    return best


def _points(coords, lo, hi):
    """Centres (metres) of voxels lo..hi-1 per axis of each block: [n][z][y][x][3]."""
    a = torch.arange(lo, hi, device=coords.device, dtype=torch.float32) + 0.5
    z, y, x = torch.meshgrid(a, a, a, indexing="ij")
    return (coords[:, None, None, None, :].float() * 8 + torch.stack([x, y, z], -1)) * VOX


def _street_blocks(boxes):
    """Keys of the blocks within mu of a surface that is seen from the street, in the order driving down it
    allocates them (those first within 50 m of the camera first, ascending (x, y, z) within a frame)."""
    dev = boxes.device
    x, y, z = torch.meshgrid(torch.arange(-6, 6, device=dev), torch.arange(-10, 2, device=dev),
                             torch.arange(-1, int((STREET_LEN + 11) / (8 * VOX)) + 1, device=dev), indexing="ij")
    c = torch.stack([x, y, z], -1).reshape(-1, 3)
    near = torch.cat([(_distance(boxes, _points(p, 0, 8)).abs() <= MU).reshape(len(p), -1).any(1)
                      for p in c.split(4096)])
    c = c[near]
    frame = (c[:, 2] * 8 * VOX - 48.0).clamp_min(0).floor().long()
    return c[torch.argsort((frame << 30) + ((c[:, 0] + 512) << 20) + ((c[:, 1] + 512) << 10) + c[:, 2] + 512)]


def _field(dist, seed, salt):
    """Fused values and weights of voxels at the given signed distances."""
    g, out = _gen(seed, salt), torch.empty_like(dist)
    w = torch.empty_like(dist)
    step = 1 << 24
    d, fo, wo = dist.reshape(-1), out.view(-1), w.view(-1)
    for i in range(0, d.numel(), step):
        p = d[i:i + step]
        rnd = torch.rand(p.shape, generator=g, device=p.device)
        seen = (p >= -MU) & (rnd > 0.03)
        f = (p / MU + 0.15 * torch.randn(p.shape, generator=g, device=p.device)).clamp(-1, 1)
        f = torch.where(p > 1.5 * MU, torch.ones_like(f), f)
        fo[i:i + step] = torch.where(seen, f, torch.zeros_like(f))
        wo[i:i + step] = torch.where(seen, torch.floor(1 + 30 * rnd * rnd), torch.zeros_like(f))
    return out, w


def _map(n, seed):
    """A fused map of n blocks: coords int32 [n][3], f and w float [n][512], and the field without its noise."""
    boxes = _boxes(seed)
    one = _street_blocks(boxes)
    reps = -(-n // len(one))
    shift = torch.zeros((reps, 1, 3), dtype=torch.long, device=one.device)
    shift[:, 0, 0] = torch.arange(reps, device=one.device) * COPY_PITCH
    coords = (one[None] + shift).reshape(-1, 3)[:n]
    dist = torch.cat([_distance(boxes, _points(p, 0, 8)).reshape(len(p), 512) for p in one.split(4096)])
    dist = dist.repeat(reps, 1)[:n]
    f, w = _field(dist, seed, 3)
    return coords.to(torch.int32).contiguous(), f, w, dist


def _volume(coords, f, w, state16=False):
    n = len(coords)
    v = D.Volume(VOX, MU, 50.0, n, max(8, int(math.ceil(math.log2(n))) + 1), 4096, max_points=0,
                 max_candidates=max(n, 64), state16=state16)
    v.insert_blocks(coords, keep_order=True)
    v.load_fused(f, w)
    return v


def _tiles(case, seed):
    """Network tiles of sampled street blocks, dual targets and their mask."""
    n, dev = case["tiles"], _dev()
    boxes, g = _boxes(seed), _gen(seed, 5)
    c = _street_blocks(boxes)
    c = c[torch.randint(len(c), (n,), generator=g, device=dev)]
    f, w = _field(torch.cat([_distance(boxes, _points(p, -1, 9)) for p in c.split(2048)]), seed, 6)
    tiles = torch.stack([f, (1.0 + w).log() / math.log(101.0)], 1).contiguous()
    fc, wc = f[:, 1:9, 1:9, 1:9], w[:, 1:9, 1:9, 1:9]
    grad = torch.tanh(4 * (f[:, 1:9, 1:9, 2:10] - fc))
    mask = ((wc > 0) & (w[:, 1:9, 1:9, 2:10] > 0)).float()
    return tiles, grad.reshape(n, 512).contiguous(), mask.reshape(n, 512).contiguous()


def _weights():
    w = warmstart.load_default_weights()
    return torch.from_numpy(warmstart.init_params(0) if w is None else w).to(_dev())


def _batch_sizes(case):
    rng = np.random.default_rng([case["volumes"], case["lo"], case["hi"]])
    return [int(round(math.exp(v))) for v in rng.uniform(math.log(case["lo"]), math.log(case["hi"]), case["volumes"])]


def _regularised(dist, w, seed):
    """The field as the surface extraction meets it: the noise nearly gone."""
    g = _gen(seed, 8)
    u = (dist / MU + 0.03 * torch.randn(dist.shape, generator=g, device=dist.device)).clamp(-1, 1)
    return torch.where(w > 0, u, torch.zeros_like(u))


def _room(rows, *shape, dtype=torch.float32):
    return torch.zeros((rows,) + shape, dtype=dtype, device=_dev())


def _map_rooms():
    return _room(ROOM, 3, dtype=torch.int32), _room(ROOM, 512), _room(ROOM, 512)


def _surface_rooms(case):
    """Rows of the arrays for a surface's points and triangles."""
    return 4096 + 64 * case["blocks"], 8192 + 300 * case["blocks"]


def _keep(room, part):
    """A session's own array with what was read back at its head."""
    room[:len(part)].copy_(part)
    return room


# ------------------------------------------------------------- prepare and run
def prepare(case, seed):
    kind = case["kind"]
    if kind == "depth":
        maps = _depth_maps(case, seed)
        fx, fy, cx, cy, w, h = _camera(case)
        vol = D.Volume(case["voxel"], 3 * case["voxel"], case["max_depth"], 1 << 15, 16, 1024, max_points=w * h,
                       state16=False)
        return {"kind": kind, "vol": vol, "rooms": _map_rooms(), "maps": maps, "K": D.intrinsics(fx, fy, cx, cy, w, h),
                "poses": [_pose(k) for k in range(len(maps))]}
    if kind == "laser":
        scans = _scans(case, seed)
        n, mu = case["rings"] * case["azimuths"], 3 * case["voxel"]
        vol = D.Volume(case["voxel"], mu, case["max_depth"], 1 << 14, 16, 1024, max_points=n, state16=False,
                       max_observations=D.laser_observations_bound(n, case["voxel"], mu, case["max_depth"]))
        return {"kind": kind, "vol": vol, "rooms": _map_rooms(), "scans": scans,
                "poses": [_pose(5 * k) for k in range(len(scans))]}
    if kind == "reg":
        vol = _volume(*_map(case["blocks"], seed)[:3], state16=case["storage"] != "f32")
        gap = case["gap_every"]
        prm = D.reg_params(LAM, STEP, STEP, iters=case["iters"], gap_every=gap, gap_tol=1e-3 if gap else 0.0,
                           storage=STORAGE[case["storage"]], gamma=case["gamma"],
                           data_term=D.DN_DATA_L1 if case["data"] == "l1" else D.DN_DATA_L2)
        return {"kind": kind, "vol": vol, "prm": prm}
    if kind == "batch":
        sizes = _batch_sizes(case)
        coords, f, w, _ = _map(max(sizes), seed)
        vols = [_volume(coords[:n].contiguous(), f[:n].contiguous(), w[:n].contiguous()) for n in sizes]
        prm = D.reg_params(LAM, STEP, STEP, iters=case["iters"], gamma=case["gamma"],
                           data_term=D.DN_DATA_L1 if case["data"] == "l1" else D.DN_DATA_L2)
        return {"kind": kind, "vols": vols, "prm": prm}
    if kind == "surface":
        coords, f, w, dist = _map(case["blocks"], seed)
        vol = _volume(coords, f, w)
        vol.regularize(D.reg_params(LAM, iters=0, init=D.DN_INIT_GIVEN, kernel=D.DN_K_FUSED),
                       u0=_regularised(dist, w, seed))
        points, triangles = _surface_rooms(case)
        return {"kind": kind, "vol": vol, "points": _room(points, 3), "mesh": _room(triangles, 3, 3)}
    if kind == "warm":
        return {"kind": kind, "vol": _volume(*_map(case["blocks"], seed)[:3]), "weights": _weights()}
    if kind == "train":
        tiles, targets, mask = _tiles(case, seed)
        g = _gen(seed, 7)
        p = _weights()
        m = 1e-3 * torch.randn(p.shape, generator=g, device=p.device)
        v = 1e-5 * (0.2 + torch.rand(p.shape, generator=g, device=p.device))
        return {"kind": kind, "tiles": tiles, "targets": targets, "mask": mask, "loss_kind": case["loss_kind"],
                "checkpoint": torch.stack([p, m, v]).contiguous(), "grad": torch.empty_like(p)}
    tiles, _, _ = _tiles(case, seed)
    return {"kind": kind, "tiles": tiles, "weights": _weights(),
            "out": torch.empty((case["tiles"], 10, 10, 10), device=_dev())}


def run(state):
    kind = state["kind"]
    if kind in ("depth", "laser"):
        vol = state["vol"]
        vol.clear()
        if kind == "depth":
            new = [vol.integrate(d, state["K"], T) for d, T in zip(state["maps"], state["poses"])]
        else:
            new = [vol.integrate_laser(p, T) for p, T in zip(state["scans"], state["poses"])]
        parts = [_keep(room, vol.extract(x)) for room, x in zip(state["rooms"], (D.DN_X_COORDS, D.DN_X_F, D.DN_X_W))]
        return {"new": new, "coords": parts[0], "f": parts[1], "w": parts[2]}
    if kind == "reg":
        vol = state["vol"]
        st = vol.regularize(state["prm"])
        return {"energy": st.energy, "dual": st.dual, "iters": st.iters_run, "u": vol.extract(D.DN_X_U),
                "p": vol.extract(D.DN_X_P)}
    if kind == "batch":
        stats = D.regularize_batch(state["vols"], state["prm"])
        return {"energy": [s.energy for s in stats], "u": [v.extract(D.DN_X_U) for v in state["vols"]]}
    if kind == "surface":
        vol = state["vol"]
        area, n = vol.mesh_area()
        return {"points": _keep(state["points"], vol.extract(D.DN_X_SURFACE)),
                "mesh": _keep(state["mesh"], vol.extract(D.DN_X_MESH)), "area": area, "triangles": n}
    if kind == "warm":
        u0, p0 = warmstart.warm_state(state["vol"], state["weights"])
        return {"u0": u0, "p0": p0}
    if kind == "train":
        pmv = state["checkpoint"].clone()   # one step on from a checkpoint
        p, m, v = pmv[0], pmv[1], pmv[2]
        loss = D.net_loss_grad(state["tiles"], p, state["targets"], state["mask"], state["grad"],
                               kind=state["loss_kind"])
        D.net_adam(p, state["grad"], m, v, 2e-4, 101)
        return {"loss": loss, "grad": state["grad"], "params": p, "m": m, "v": v}
    D.net_forward(state["tiles"], state["weights"], state["out"])
    return state["out"]


def work(case):
    kind = case["kind"]
    if kind == "depth":
        px = case["width"] * case["height"] * case["frames"]
        return {"bytes": 4 * px + 8 * 512 * 1500, "flops": 100 * px}
    if kind == "laser":
        n = case["rings"] * case["azimuths"] * case["scans"]
        obs = n * 0.4 * case["max_depth"] / case["voxel"]   # voxels along the rays
        return {"bytes": 12 * n + 8 * 512 * 1500, "flops": 20 * obs}
    if kind == "reg":
        vox = 512 * case["blocks"]
        return {"bytes": 24 * vox, "flops": 45 * vox * case["iters"]}   # f, w read; u, p written
    if kind == "batch":
        lo, hi = case["lo"], case["hi"]
        vox = 512 * case["volumes"] * (hi - lo) / math.log(hi / lo)     # the mean of the sizes' distribution
        return {"bytes": 12 * vox, "flops": 45 * vox * case["iters"]}
    if kind == "surface":
        vox = 512 * case["blocks"]
        return {"bytes": 5 * vox + 8000 * case["blocks"], "flops": 20 * vox}   # about 220 triangles a block
    if kind == "warm":
        vox = 512 * case["blocks"]
        return {"bytes": 24 * vox, "flops": 3 * 15.99e6 * case["blocks"]}
    if kind == "train":
        return {"bytes": 4 * case["tiles"] * 3024 + 4 * 8241 * 8, "flops": 47.52e6 * case["tiles"]}
    return {"bytes": 12000 * case["tiles"] + 4 * 8241, "flops": 20.5e6 * case["tiles"]}


# ------------------------------------------------ what 64 bits give (no library)
_OFF = 1 << 20


def _keys(c):
    c = c.long() + _OFF
    return (c[..., 0] << 42) | (c[..., 1] << 21) | c[..., 2]


class _Lookup:
    """Block keys -> pool ids (-1: not there)."""

    def __init__(self, coords):
        self.keys, self.ids = torch.sort(_keys(coords))

    def __call__(self, c):
        k = _keys(c)
        i = torch.searchsorted(self.keys, k).clamp_max(len(self.keys) - 1)
        return torch.where(self.keys[i] == k, self.ids[i], torch.full_like(i, -1))


def _walk(a, b, limit):
    """The cells of the unit grid that segments a -> b (float64 [n][3]) pass, one step at a time: (cell, alive)."""
    alive = ((a.abs() < limit) & (b.abs() < limit)).all(1)
    a = torch.where(alive[:, None], a, torch.zeros_like(a))
    b = torch.where(alive[:, None], b, torch.zeros_like(b))
    k, e = a.floor(), b.floor()
    step, left = torch.sign(e - k), (e - k).abs()
    d = torch.where(step == 0, torch.ones_like(a), b - a)
    zero = torch.zeros_like(a)
    tmax = torch.where(step > 0, (k + 1 - a) / d, torch.where(step < 0, (k - a) / d, zero))
    tdel = torch.where(step == 0, zero, step / d)
    inf = torch.full_like(a, math.inf)
    while True:
        yield k, alive
        t = torch.where(left > 0, tmax, inf)
        best, c = t[:, 0], torch.zeros(len(a), dtype=torch.long, device=a.device)
        for i in (1, 2):
            less = t[:, i] < best
            best, c = torch.where(less, t[:, i], best), torch.where(less, torch.full_like(c, i), c)
        alive = alive & (left > 0).any(1)
        if not bool(alive.any()):
            return
        one = torch.nn.functional.one_hot(c, 3).bool() & alive[:, None]
        k, tmax = torch.where(one, k + step, k), torch.where(one, tmax + tdel, tmax)
        left = torch.where(one, left - 1, left)


def _over(x, s):
    """x / s, rounded once (torch multiplies by the reciprocal of a number that it is given as one)."""
    return x / torch.tensor(s, dtype=F64, device=x.device)


def _affine(T, p):
    return torch.stack([((T[i, 0] * p[:, 0] + T[i, 1] * p[:, 1]) + T[i, 2] * p[:, 2]) + T[i, 3] for i in range(3)], 1)


def _new_blocks(cells, coords):
    """The cells' keys that coords does not hold, ascending."""
    k = torch.unique(_keys(cells))
    if len(coords):
        k = k[~torch.isin(k, _keys(coords))]
    m = (1 << 21) - 1
    return torch.stack([((k >> 42) & m) - _OFF, ((k >> 21) & m) - _OFF, (k & m) - _OFF], 1)


def _grow(coords, f, w, cells):
    fresh = _new_blocks(cells, coords)
    z = torch.zeros((len(fresh), 512), dtype=F64, device=f.device)
    return torch.cat([coords, fresh]), torch.cat([f, z]), torch.cat([w, z.clone()]), len(fresh)


def _band_cells(a, b, bs, limit):
    return torch.cat([k[alive].long() for k, alive in _walk(_over(a, bs), _over(b, bs), limit)])


def _session(new, coords, f, w):
    return {"new": new, "coords": _keep(_room(ROOM, 3, dtype=torch.int32), coords.to(torch.int32)),
            "f": _keep(_room(ROOM, 512, dtype=F64), f), "w": _keep(_room(ROOM, 512, dtype=F64), w)}


def _exact_fusion(case, seed):
    dev, s, mu, far = _dev(), case["voxel"], 3 * case["voxel"], case["max_depth"]
    coords = torch.zeros((0, 3), dtype=torch.long, device=dev)
    f = torch.zeros((0, 512), dtype=F64, device=dev)
    w = f.clone()
    new = []
    v = torch.arange(512, device=dev)
    local = torch.stack([v & 7, (v >> 3) & 7, v >> 6], 1)
    if case["kind"] == "depth":
        fx, fy, cx, cy, W, H = _camera(case)
        px = torch.arange(W * H, device=dev)
        rx, ry = _over((px % W).double() - cx, fx), _over((px // W).double() - cy, fy)
        for k, depth in enumerate(_depth_maps(case, seed)):
            T = torch.from_numpy(_pose(k)).to(dev)
            d = depth.reshape(-1).double()
            ok = torch.isfinite(d) & (d > 0) & (d <= far)
            z0, z1 = (d - mu).clamp_min(1e-3), d + mu
            a = _affine(T, torch.stack([z0 * rx, z0 * ry, z0], 1))[ok]
            b = _affine(T, torch.stack([z1 * rx, z1 * ry, z1], 1))[ok]
            coords, f, w, n = _grow(coords, f, w, _band_cells(a, b, 8 * s, 1e6))
            new.append(n)
            for i in range(0, len(coords), 8192):
                q = ((8 * coords[i:i + 8192, None, :] + local).double() + 0.5) * s - T[:3, 3]
                xc, yc, zc = (((T[0, j] * q[..., 0] + T[1, j] * q[..., 1]) + T[2, j] * q[..., 2]) for j in range(3))
                X, Y = fx * (xc / zc) + cx + 0.5, fy * (yc / zc) + cy + 0.5
                hit = (zc > 0) & (X >= 0) & (X < W) & (Y >= 0) & (Y < H)
                at = torch.where(hit, Y.floor() * W + X.floor(), torch.zeros_like(X)).long()
                eta = d[at] - zc
                hit &= ok[at] & (eta >= -mu)
                fo, wo = f[i:i + 8192], w[i:i + 8192]
                psi = (eta / mu).clamp_max(1.0)
                f[i:i + 8192] = torch.where(hit, (psi + wo * fo) / (wo + 1), fo)
                w[i:i + 8192] = torch.where(hit, wo + 1, wo)
        return _session(new, coords, f, w)
    for k, pts in enumerate(_scans(case, seed)):
        T = torch.from_numpy(_pose(5 * k)).to(dev)
        p = pts.double()
        p = p[torch.isfinite(p).all(1)]
        r = torch.sqrt((p[:, 0] * p[:, 0] + p[:, 1] * p[:, 1]) + p[:, 2] * p[:, 2])
        ok = (r > 0) & (r <= far)
        p, r = p[ok], r[ok]
        d = p / r[:, None]
        near, end = (r - mu).clamp_min(1e-3), r + mu
        coords, f, w, n = _grow(coords, f, w, _band_cells(_affine(T, near[:, None] * d), _affine(T, end[:, None] * d),
                                                          8 * s, 1e9))
        new.append(n)
        find = _Lookup(coords)
        total, count = torch.zeros(len(coords) * 512, dtype=F64, device=dev), torch.zeros(len(coords) * 512, dtype=F64,
                                                                                      device=dev)
        Dw = torch.stack([(T[i, 0] * d[:, 0] + T[i, 1] * d[:, 1]) + T[i, 2] * d[:, 2] for i in range(3)], 1)
        for c, alive in _walk(_over(_affine(T, 0.0 * d), s), _over(_affine(T, end[:, None] * d), s), 1e9):
            cell = c.long()
            b = find(cell >> 3)
            rho = torch.zeros_like(r)
            for i in range(3):
                rho = rho + ((c[:, i] + 0.5) * s - T[i, 3]) * Dw[:, i]
            eta = r - rho
            hit = alive & (b >= 0) & (eta >= -mu)
            lo = cell & 7
            at = (b * 512 + lo[:, 0] + 8 * lo[:, 1] + 64 * lo[:, 2])[hit]
            total.index_add_(0, at, (eta / mu).clamp_max(1.0)[hit])
            count.index_add_(0, at, torch.ones_like(at, dtype=F64))
        total, count = total.reshape(-1, 512), count.reshape(-1, 512)
        f = torch.where(count > 0, (w * f + total) / (w + count).clamp_min(1), f)
        w = w + count
    return _session(new, coords, f, w)


def _neighbours(coords):
    """Flat voxel index of g + e_a and of g - e_a for each axis ([3][n * 512]; n * 512 where there is none)."""
    n, dev = len(coords), coords.device
    find, none = _Lookup(coords), n * 512
    v = torch.arange(512, device=dev)
    l3 = torch.stack([v & 7, (v >> 3) & 7, v >> 6], 1)
    base = torch.arange(n, device=dev)[:, None] * 512
    up, down = [], []
    for a, stride in enumerate((1, 8, 64)):
        e = torch.zeros(3, dtype=torch.long, device=dev)
        e[a] = 1
        for sign, edge, out in ((1, 7, up), (-1, 0, down)):
            b = find(coords.long() + sign * e)[:, None]
            over = torch.where(b >= 0, b * 512 + v - sign * 7 * stride, torch.full_like(b, none))
            out.append(torch.where(l3[:, a] == edge, over, base + v + sign * stride).reshape(-1))
    return up, down


def _at(x, i):
    return torch.cat([x, x.new_zeros(1)])[i]


def _exact_solve(coords, f, w, prm, l1, gamma, gap_every):
    """Chambolle-Pock on the masked energy in float64: u, p, E, D, iterations."""
    f, w = f.reshape(-1).double(), w.reshape(-1).double()
    up, down = _neighbours(coords)
    om = w > 0
    m = [om & _at(om, i).bool() for i in up]
    u, ub = torch.zeros_like(f), torch.zeros_like(f)
    p = [torch.zeros_like(f) for _ in range(3)]
    tau, sigma, theta = STEP, STEP, 1.0

    def div():
        d = torch.zeros_like(f)
        for a in range(3):
            q = torch.where(m[a], p[a], torch.zeros_like(f))
            d += q - _at(q, down[a])
        return d

    def energies():
        g = [torch.where(m[a], _at(u, up[a]) - u, torch.zeros_like(u)) for a in range(3)]
        tv = torch.sqrt((g[0] * g[0] + g[1] * g[1]) + g[2] * g[2])
        d = div()
        if l1:
            e = tv + LAM * w * (u - f).abs()
            q = torch.minimum(torch.minimum(-f * d, -d + LAM * w * (1 - f).abs()), d + LAM * w * (1 + f).abs())
        else:
            e = tv + 0.5 * LAM * w * (u - f).square()
            q = -f * d - d * d / (2 * LAM * w)
        return float(e[om].sum()), float(q[om].sum())

    it = 0
    while it < prm:
        if gamma > 0:
            theta = 1.0 / math.sqrt(1.0 + 2.0 * gamma * tau)
        for a in range(3):
            p[a] += sigma * torch.where(m[a], _at(ub, up[a]) - ub, torch.zeros_like(ub))
        n = torch.sqrt((p[0] * p[0] + p[1] * p[1]) + p[2] * p[2]).clamp_min(1.0)
        for a in range(3):
            p[a] /= n
        ut = u + tau * div()
        tlw = tau * LAM * w
        if l1:
            r = ut - f
            nu = (f + torch.sign(r) * (r.abs() - tlw).clamp_min(0)).clamp(-1, 1)
        else:
            nu = (ut + tlw * f) / (1 + tlw)
        nu = torch.where(om, nu, u)
        ub, u = nu + theta * (nu - u), nu
        if gamma > 0:
            tau, sigma = theta * tau, sigma / theta
        it += 1
        if gap_every and it % gap_every == 0 and it < prm:
            e, d = energies()
            if e - d <= 1e-3 * e:
                break
    e, d = energies()
    return u.reshape(-1, 512), torch.stack(p).reshape(3, -1, 512), e, d, it


_AXES = ((0, 1), (0, 2), (1, 0), (1, 2), (2, 0), (2, 1))


def _exact_surface(case, seed):
    coords, _, w, dist = _map(case["blocks"], seed)
    u = _regularised(dist, w, seed).reshape(-1).double()
    up, _ = _neighbours(coords)
    om = w.reshape(-1) > 0
    n, dev = len(u), u.device
    v = torch.arange(512, device=dev)
    cell = (coords.long()[:, None, :] * 8 + torch.stack([v & 7, (v >> 3) & 7, v >> 6], 1)).reshape(-1, 3)
    neg = u < 0
    cross = torch.stack([om & _at(om, i).bool() & (neg != _at(neg, i).bool()) for i in up], 1)
    g, a = torch.nonzero(cross, as_tuple=True)
    u0, u1 = u[g], torch.stack([_at(u, i) for i in up], 1)[g, a]
    pts = (cell[g].double() + 0.5) * VOX
    pts[torch.arange(len(g), device=dev), a] += u0 / (u0 - u1) * VOX
    # the eight corners of every cube, its six tetrahedra and their triangles
    corner = [torch.arange(n, device=dev)]
    for a in range(3):
        ext = torch.cat([up[a], up[a].new_full((1,), n)])
        corner = corner + [ext[c] for c in corner]
    full = torch.ones_like(om)
    for c in corner:
        full &= _at(om, c).bool()
    cube = torch.nonzero(full).flatten()
    cu = torch.stack([u[c[cube]] for c in corner], 1)
    base = cell[cube].double()
    kk = torch.tensor([[0, 1 << a0, (1 << a0) | (1 << a1), 7] for a0, a1 in _AXES], device=dev)
    offs = torch.tensor([[k & 1, (k >> 1) & 1, k >> 2] for k in range(8)], dtype=F64, device=dev)
    tu = cu[:, kk]                                        # [cubes][6][4]
    tn = tu < 0
    nneg = tn.sum(-1)
    cid, tid = torch.nonzero((nneg > 0) & (nneg < 4), as_tuple=True)
    tn, nneg, kt, cu, base = tn[cid, tid], nneg[cid, tid], kk[tid], cu[cid], base[cid]
    order = torch.argsort((~tn).long() * 4 + torch.arange(4, device=dev), 1)      # negatives first, ascending
    two = nneg == 2
    first = torch.where(nneg == 3, 3, 0)                   # where the vertex alone on its side stands
    odd = order.gather(1, first[:, None])[:, 0]
    rest = torch.argsort((torch.arange(4, device=dev) == odd[:, None]).long() * 8 + torch.arange(4, device=dev), 1)
    a, b, c, d = order[:, 0], order[:, 1], order[:, 2], order[:, 3]
    tri1 = torch.where(two[:, None], torch.stack([a, c, a, d, b, d], 1),
                       torch.stack([odd, rest[:, 0], odd, rest[:, 1], odd, rest[:, 2]], 1))
    tri2 = torch.stack([a, c, b, d, b, c], 1)
    pick = torch.cat([torch.arange(len(cid), device=dev) * 2, torch.nonzero(two).flatten() * 2 + 1])
    edges = torch.cat([tri1, tri2[two]])
    src = torch.cat([torch.arange(len(cid), device=dev), torch.nonzero(two).flatten()])
    by = torch.argsort(pick)
    edges, src = edges[by], src[by]
    ks = kt[src].gather(1, edges).reshape(-1, 3, 2)
    ks = torch.sort(ks, -1).values
    uu = cu[src].gather(1, ks.reshape(-1, 6)).reshape(-1, 3, 2)
    t = uu[..., 0] / (uu[..., 0] - uu[..., 1])
    p0 = (base[src][:, None] + offs[ks[..., 0]] + 0.5) * VOX
    p1 = (base[src][:, None] + offs[ks[..., 1]] + 0.5) * VOX
    tri = p0 + t[..., None] * (p1 - p0)
    cr = torch.linalg.cross(tri[:, 1] - tri[:, 0], tri[:, 2] - tri[:, 0])
    oc, tv = offs[kt], tn[..., None].double()
    r = ((1 - tv) * oc).sum(1) * nneg[:, None].double() - (tv * oc).sum(1) * (4 - nneg)[:, None].double()
    flip = (cr * r[src]).sum(1) < 0
    tri[flip] = tri[flip][:, [0, 2, 1]]
    points, triangles = _surface_rooms(case)
    return {"points": _keep(_room(points, 3, dtype=F64), pts), "mesh": _keep(_room(triangles, 3, 3, dtype=F64), tri),
            "area": float(0.5 * cr.square().sum(1).sqrt().sum()), "triangles": len(tri)}


def _conv(x, w, b):
    """3^3 convolution with zero padding: x [B][ci][10][10][10], w [co][ci][27]."""
    xp = torch.nn.functional.pad(x, (1, 1, 1, 1, 1, 1))
    y = 0
    for t in range(27):
        kx, ky, kz = t % 3, (t // 3) % 3, t // 9
        y = y + torch.tensordot(w[:, :, t].contiguous(), xp[:, :, kz:kz + 10, ky:ky + 10, kx:kx + 10], ([1], [1]))
    return y.transpose(0, 1) + b.reshape(1, -1, 1, 1, 1)


def _net(x, p):
    h = torch.relu(_conv(x, p[0:864].reshape(16, 2, 27), p[864:880]))
    h = torch.relu(_conv(h, p[880:7792].reshape(16, 16, 27), p[7792:7808]))
    return _conv(h, p[7808:8240].reshape(1, 16, 27), p[8240:8241])[:, 0]


def _exact_warm(case, seed):
    coords, f, w, _ = _map(case["blocks"], seed)
    n, dev, p = len(coords), coords.device, _weights().double()
    find = _Lookup(coords)
    fd, wd = f.reshape(-1).double(), torch.log(1 + w.reshape(-1).double()) / math.log(101.0)
    up, _ = _neighbours(coords)
    om = w.reshape(-1) > 0
    ax = torch.arange(-1, 9, device=dev)
    z, y, x = torch.meshgrid(ax, ax, ax, indexing="ij")
    cell = torch.stack([x, y, z], -1)
    out = torch.zeros((3, n, 512), dtype=F64, device=dev)
    for i in range(0, n, 512):
        c = coords[i:i + 512].long()[:, None, None, None, :] * 8 + cell
        b = find(c >> 3)
        lo = c & 7
        at = torch.where(b >= 0, b * 512 + lo[..., 0] + 8 * lo[..., 1] + 64 * lo[..., 2], torch.full_like(b, n * 512))
        tile = torch.stack([_at(fd, at), _at(wd, at)], 1)
        for a, dims in enumerate(((0, 1, 2, 3, 4), (0, 1, 2, 4, 3), (0, 1, 4, 3, 2))):
            r = _net(tile.permute(dims), p)[:, None].permute(dims)[:, 0]
            out[a, i:i + 512] = r[:, 1:9, 1:9, 1:9].reshape(-1, 512)
    out = torch.where(torch.stack([om & _at(om, i).bool() for i in up]).reshape(3, n, 512), out, torch.zeros_like(out))
    nrm = torch.sqrt((out[0] * out[0] + out[1] * out[1]) + out[2] * out[2]).clamp_min(1.0)
    return {"u0": torch.where(w > 0, f, torch.zeros_like(f)).double(), "p0": out / nrm}


def _exact_train(case, seed):
    s = prepare(case, seed)
    p, m, v = s["checkpoint"].double()
    p = p.clone().requires_grad_(True)
    x = s["tiles"].double()
    pred = torch.cat([_net(t, p) for t in x.split(128)])[:, 1:9, 1:9, 1:9].reshape(-1, 512)
    if s["loss_kind"] == 0:
        pred = pred + x[:, 0, 1:9, 1:9, 1:9].reshape(-1, 512)
    mask = s["mask"].double()
    loss = (mask * (pred - s["targets"].double()).square()).sum() / mask.sum().clamp_min(1.0)
    loss.backward()
    g = p.grad
    m, v = 0.9 * m + 0.1 * g, 0.999 * v + 0.001 * g * g
    q = p.detach() - 2e-4 * (m / (1 - 0.9 ** 101)) / (torch.sqrt(v / (1 - 0.999 ** 101)) + 1e-8)
    return {"loss": float(loss.detach()), "grad": g, "params": q, "m": m, "v": v}


def exact(case, seed):
    kind = case["kind"]
    if kind in ("depth", "laser"):
        return _exact_fusion(case, seed)
    if kind == "reg":
        if case["blocks"] * case["iters"] > 6.2e6:
            return None
        u, p, e, d, it = _exact_solve(*_map(case["blocks"], seed)[:3], case["iters"], case["data"] == "l1",
                                      case["gamma"], case["gap_every"])
        if case["storage"] != "f32" and case["gap_every"]:
            return None      # rounding to 16 bits moves the iteration that stops it
        return {"energy": e, "dual": d, "iters": it, "u": u, "p": p}
    if kind == "batch":
        coords, f, w, _ = _map(max(_batch_sizes(case)), seed)
        got = [_exact_solve(coords[:n], f[:n], w[:n], case["iters"], case["data"] == "l1", case["gamma"], 0)
               for n in _batch_sizes(case)]
        return {"energy": [g[2] for g in got], "u": [g[0] for g in got]}
    if kind == "surface":
        return _exact_surface(case, seed)
    if kind == "warm":
        return _exact_warm(case, seed)
    if kind == "train":
        return _exact_train(case, seed)
    s = prepare(case, seed)
    return torch.cat([_net(t, s["weights"].double()) for t in s["tiles"].double().split(128)])

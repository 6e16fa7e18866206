"""Performance cases of the LiDAR engine: what a simulation program asks of it per frame.

A case is a dict of plain values.  ``listed()`` names twelve that span the range of use: a small sensor's frame
(latency), ordinary and ragged frames, the scanning sensor's full frame, the range-corrected option, a pinhole
rendering, the stateless call, batches of small and of mixed frames, the surrogate network's forward pass, its
gradients, a surrogate frame and range stacking.  ``draw(rng)`` gives further cases of the same ranges.
``prepare`` renders a seeded synthetic G-buffer on the GPU and builds the handle that a program keeps; ``run`` is
one pass through the public entry points with the results read into device tensors; ``work`` counts the bytes and
operations a pass cannot do without; ``exact`` gives the outputs in 64 bits from plain torch.
"""
import math
from types import SimpleNamespace

import numpy as np
import torch

import paper_2512_05932_amd as lidar

LIGHT = 299792458.0
ROAD_THRESHOLD = 9.345e-08          # detection threshold and sun of the scanning sensor
ROAD_SUN = 0.02841
SENSOR_HEIGHT = 0.5
SUR_LAYERS = ((1056, 256), (256, 256), (256, 256), (256, 16))
SUR_PARAMS = sum(i * o + o for i, o in SUR_LAYERS)

# echo selections and range modes by the names used in the cases
SELECT = {"all": lidar.LIDAR_ECHO_ALL, "strongest": lidar.LIDAR_ECHO_STRONGEST,
          "raw_nearest": lidar.LIDAR_ECHO_RAW_NEAREST}
RANGES = {"centre": lidar.LIDAR_RANGE_CENTRE, "corrected": lidar.LIDAR_RANGE_CORRECTED}

FRAME = {"kind": "frame", "scene": "road", "width": 1024, "height": 512, "fov_az": 60.0, "fov_el": 30.0,
         "steer": "grid", "n_az": 40, "n_el": 25, "pattern": "gauss", "sigma_az": 0.1, "sigma_el": 0.1,
         "bins": 2048, "bin_ns": 0.5, "select": "all", "range": "centre"}


def listed():
    return [
        # the smallest sensor: 40 x 25 narrow beams over random surfaces; launches and latency count
        {**FRAME, "name": "frame-small", "scene": "iid", "bins": 512, "bin_ns": 1.0},
        # an odd raster, Lissajous steering, a middle footprint, one (the strongest) echo per beam
        {**FRAME, "name": "frame-ragged", "width": 1501, "height": 333, "steer": "lissajous", "n_az": 7001, "n_el": 1,
         "sigma_az": 0.181, "sigma_el": 0.409, "bins": 1200, "bin_ns": 1.0, "select": "strongest"},
        # the scanning sensor: 16 x 1800 beams with wide pattern tails and the sun's floor (the benchmark's frame)
        {**FRAME, "name": "frame-scan", "width": 8192, "fov_az": 145.0, "fov_el": 3.2, "n_az": 1800, "n_el": 16,
         "pattern": "table"},
        # ranges corrected for every sample with the surface normal (a smaller scan)
        {**FRAME, "name": "frame-corrected", "width": 4096, "height": 256, "fov_az": 145.0, "fov_el": 3.2, "n_az": 900,
         "n_el": 16, "pattern": "table", "range": "corrected"},
        # a rasteriser's pinhole image with a 24-bit z buffer, reprojected and simulated
        {**FRAME, "name": "frame-pinhole", "kind": "pinhole", "width": 4096, "height": 1024, "fov_az": 90.0,
         "fov_el": 45.0, "n_az": 500, "n_el": 64, "sigma_az": 0.0425, "sigma_el": 0.085, "src_w": 1920, "src_h": 1080},
        # the call that keeps no state and allocates nothing: a new steering pattern with every frame
        {**FRAME, "name": "static-frame", "kind": "static", "n_az": 100, "n_el": 50, "steer": "jitter"},
        # a rig of eight small sensors replayed as one graph
        {**FRAME, "name": "batch-rig", "kind": "batch", "frames": 8, "mixed": False, "scene": "iid", "bins": 512,
         "bin_ns": 1.0},
        # sensors of very different sizes in one batch (both scenes, 20 to 20000 pixel footprints)
        {**FRAME, "name": "batch-mixed", "kind": "batch", "frames": 12, "mixed": True, "width": 2048, "height": 1024,
         "n_az": 160, "n_el": 100},
        # the surrogate network alone: a scan's beams, and its loss gradients on a training minibatch
        {"name": "surrogate-forward", "kind": "forward", "rows": 128000},
        {"name": "surrogate-gradients", "kind": "gradients", "rows": 4096},
        # a whole frame in surrogate mode: inputs, network, gate and the plain path for the rejected beams
        {**FRAME, "name": "surrogate-frame", "kind": "surrogate", "width": 8192, "fov_az": 145.0, "fov_el": 3.2,
         "n_az": 2000, "n_el": 64, "sigma_az": 0.0425, "sigma_el": 0.34},
        # the slice-by-slice algorithm on a whole image
        {"name": "range-stacking", "kind": "stack", "width": 4096, "height": 512, "fov_az": 145.0, "fov_el": 12.8,
         "M": 34, "N": 41, "core_az": 0.0425, "core_el": 0.34, "bins": 1200, "bin_ns": 1.0},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("frame", "frame", "frame", "pinhole", "static", "batch", "batch", "forward", "gradients",
                       "surrogate", "stack"))
    if kind == "forward":
        return {"kind": kind, "rows": _log(rng, 48, 128000)}
    if kind == "gradients":
        return {"kind": kind, "rows": _log(rng, 64, 8192)}
    if kind == "stack":
        w, h = _log(rng, 256, 4096), _log(rng, 64, 512)
        return {"kind": kind, "width": w, "height": h, "fov_az": 145.0, "fov_el": 12.8, "M": _log(rng, 3, 34),
                "N": _log(rng, 3, 41), "core_az": 0.0425, "core_el": 0.34, "bins": rng.choice((512, 1200)),
                "bin_ns": 1.0}
    c = dict(FRAME, kind=kind)
    c["scene"] = rng.choice(("road", "iid"))
    c["bins"], c["bin_ns"] = rng.choice(((512, 1.0), (1200, 1.0), (2048, 0.5)))
    if kind == "surrogate":
        c.update(scene="road", bins=2048, bin_ns=0.5, width=_log(rng, 1024, 8192), height=_log(rng, 128, 512),
                 fov_az=145.0, fov_el=3.2, n_az=_log(rng, 100, 2000), n_el=_log(rng, 8, 64), sigma_az=0.0425,
                 sigma_el=0.34)
        return c
    if kind == "batch":
        c.update(frames=rng.randint(2, 12), mixed=rng.random() < 0.6, width=_log(rng, 256, 2048),
                 height=_log(rng, 128, 1024), n_az=_log(rng, 20, 160), n_el=_log(rng, 10, 100))
        return c
    c["steer"] = rng.choice(("grid", "lissajous", "jitter"))
    c["select"] = rng.choice(("all", "all", "all", "strongest", "raw_nearest"))
    c["width"], c["height"] = _log(rng, 256, 4096), _log(rng, 64, 1024)
    n = _log(rng, 200, 20000)
    c["n_el"] = rng.choice((1, 7, 16, 32, 64)) if c["steer"] != "lissajous" else 1
    c["n_az"] = max(1, n // c["n_el"])
    if kind == "frame" and rng.random() < 0.35:
        c.update(fov_az=145.0, fov_el=3.2, pattern="table", scene="road", bins=2048, bin_ns=0.5, n_az=_log(rng, 50, 1000),
                 n_el=16, steer="grid", height=_log(rng, 64, 512))
        if rng.random() < 0.4:
            c.update(range="corrected", width=_log(rng, 512, 4096), height=_log(rng, 64, 256), n_az=_log(rng, 50, 600))
        return c
    if kind == "pinhole":
        c.update(scene="road", fov_az=90.0, fov_el=45.0, src_w=_log(rng, 320, 1920), src_h=_log(rng, 180, 1080))
    # footprint of F pixels, cut at 3 sigma
    s = math.sqrt(_log(rng, 20, 6000) / math.pi) / 3.0
    c["sigma_az"], c["sigma_el"] = s * c["fov_az"] / c["width"], s * c["fov_el"] / c["height"]
    return c


# ---- inputs ------------------------------------------------------------------------------------------------------


def _raster(c):
    return SimpleNamespace(width=c["width"], height=c["height"], az_min=-0.5 * c["fov_az"], az_max=0.5 * c["fov_az"],
                           el_min=-0.5 * c["fov_el"], el_max=0.5 * c["fov_el"])


def _angles(r):
    f64 = dict(dtype=torch.float64, device="cuda")
    az = torch.deg2rad(r.az_min + (torch.arange(r.width, **f64) + 0.5) * ((r.az_max - r.az_min) / r.width))
    el = torch.deg2rad(r.el_max - (torch.arange(r.height, **f64) + 0.5) * ((r.el_max - r.el_min) / r.height))
    return az, el


def _directions(r):
    az, el = _angles(r)
    ce = torch.cos(el)[:, None]
    return ce * torch.cos(az)[None], ce * torch.sin(az)[None], torch.sin(el)[:, None].expand(r.height, r.width)


def _iid_scene(r, seed):
    """Every pixel a surface of its own: depth, reflectance, tilt up to 60 degrees, 2 % retroreflectors."""
    g = torch.Generator("cuda").manual_seed(seed)

    def uni(lo, hi):
        return lo + (hi - lo) * torch.rand((r.height, r.width), generator=g, device="cuda", dtype=torch.float64)
    a = [-d for d in _directions(r)]
    depth, rho, cos, psi = uni(5.0, 60.0), uni(0.05, 0.9), uni(0.5, 1.0), uni(0.0, 2.0 * math.pi)
    gain = torch.where(uni(0.0, 1.0) < 0.02, 100.0, 1.0)
    # a basis orthogonal to -view: t1 horizontal, t2 = a x t1
    h = torch.sqrt(a[0] ** 2 + a[1] ** 2)
    t1 = (-a[1] / h, a[0] / h)
    t2 = (-a[2] * t1[1], a[2] * t1[0], a[0] * t1[1] - a[1] * t1[0])
    s = torch.sqrt(1.0 - cos * cos)
    sc, ss = s * torch.cos(psi), s * torch.sin(psi)
    n = (a[0] * cos + t1[0] * sc + t2[0] * ss, a[1] * cos + t1[1] * sc + t2[1] * ss, a[2] * cos + t2[2] * ss)
    return tuple(t.to(torch.float32).contiguous() for t in (depth, rho, gain, *n))


def _cast_road(d, seed, n_boxes=24):
    """Ray cast of a road plane and vehicle-like boxes with retroreflective plates along the unit directions d."""
    rng = np.random.default_rng(seed)
    inf = torch.full((), math.inf, dtype=torch.float64, device="cuda")
    depth = torch.where(d[2] < 0.0, -SENSOR_HEIGHT / torch.where(d[2] < 0.0, d[2], -1.0), inf)
    shape = depth.shape
    rho = torch.where(torch.isfinite(depth), float(rng.uniform(0.05, 0.9)), 0.0).to(torch.float64)
    gain = torch.ones(shape, dtype=torch.float64, device="cuda")
    n = [torch.zeros(shape, dtype=torch.float64, device="cuda") for _ in range(3)]
    n[2] += 1.0
    for _ in range(n_boxes):
        cx, cy, yaw = rng.uniform(5.0, 140.0), rng.uniform(-15.0, 15.0), rng.uniform(-0.3, 0.3)
        half = np.array([rng.uniform(4.0, 12.0), rng.uniform(1.8, 2.6), rng.uniform(1.4, 3.5)]) * 0.5
        b_rho, plate = rng.uniform(0.05, 0.9), rng.uniform(-0.5, 0.5)
        c, s = math.cos(yaw), math.sin(yaw)
        o = (-(c * cx + s * cy), s * cx - c * cy, SENSOR_HEIGHT - half[2])
        loc = (c * d[0] + s * d[1], c * d[1] - s * d[0], d[2])
        t_in, t_out, axis = -inf, inf, torch.zeros(shape, dtype=torch.int64, device="cuda")
        for k in range(3):
            inv = 1.0 / torch.where(loc[k].abs() < 1e-12, 1e-12, loc[k])
            ta, tb = (-half[k] - o[k]) * inv, (half[k] - o[k]) * inv
            near, far = torch.minimum(ta, tb), torch.maximum(ta, tb)
            axis = torch.where(near > t_in, k, axis)
            t_in, t_out = torch.maximum(near, t_in), torch.minimum(far, t_out)
        hit = (t_in <= t_out) & (t_in > 1e-6) & (t_in < depth)
        depth, rho = torch.where(hit, t_in, depth), torch.where(hit, b_rho, rho)
        nl = [torch.where(axis == k, -torch.sign(loc[k]), 0.0) for k in range(3)]
        for k, v in enumerate((c * nl[0] - s * nl[1], s * nl[0] + c * nl[1], nl[2])):
            n[k] = torch.where(hit, v, n[k])
        side = torch.where(axis == 0, o[1] + loc[1] * t_in, o[0] + loc[0] * t_in)
        top = o[2] + loc[2] * t_in
        on = hit & (axis != 2) & ((side - plate * half[1]).abs() < 0.3) & ((top + 0.3 * half[2]).abs() < 0.15)
        gain = torch.where(on, 500.0, torch.where(hit, 1.0, gain))
    return depth, rho, gain, n


def _planes(c, r, seed):
    if c["scene"] == "iid":
        return _iid_scene(r, seed)
    depth, rho, gain, n = _cast_road(_directions(r), seed)
    return tuple(t.to(torch.float32).contiguous() for t in (depth, rho, gain, *n))


def _pinhole(c, seed):
    """A pinhole rendering of the road scene with a 24-bit z buffer (camera frame x right, y down, z forward)."""
    w, h, near, far = c["src_w"], c["src_h"], 0.3, 1000.0
    f = 0.5 * w / math.tan(math.radians(45.0))
    pitch = math.radians(-2.0)
    rot = np.array([[math.cos(pitch), 0.0, -math.sin(pitch)], [0.0, 1.0, 0.0], [math.sin(pitch), 0.0, math.cos(pitch)]]) @ \
        np.array([[0.0, 0.0, 1.0], [-1.0, 0.0, 0.0], [0.0, -1.0, 0.0]])
    f64 = dict(dtype=torch.float64, device="cuda")
    x = ((torch.arange(w, **f64) + 0.5 - 0.5 * w) / f)[None].expand(h, w)
    y = ((torch.arange(h, **f64) + 0.5 - 0.5 * h) / f)[:, None].expand(h, w)
    norm = torch.sqrt(x * x + y * y + 1.0)
    cam = (x / norm, y / norm, 1.0 / norm)
    depth, rho, gain, n = _cast_road([sum(float(rot[i, j]) * cam[j] for j in range(3)) for i in range(3)], seed)
    z = depth / norm
    buf = torch.where(torch.isfinite(z), far * (z - near) / (z * (far - near)), 1.0).clamp(0.0, 1.0)
    q = torch.round(torch.nan_to_num(buf, nan=1.0) * 16777215.0).to(torch.int32)
    n_cam = [sum(float(rot[j, i]) * n[j] for j in range(3)) for i in range(3)]
    planes = (q,) + tuple(t.to(torch.float32).contiguous() for t in (rho, gain, *n_cam))
    return SimpleNamespace(width=w, height=h, fx=f, fy=f, cx=0.5 * w, cy=0.5 * h, rot=rot, fmt=4, near=near, far=far), planes


def _table():
    """The scanning sensor's combined pattern: an elliptic core and a weak disc tail on 256 x 256 cells over +-2 deg."""
    x = -2.0 + (np.arange(256) + 0.5) * (4.0 / 256)
    yy, xx = np.meshgrid(-x, x, indexing="ij")
    k = 1.0 / (2.0 * math.sqrt(2.0 * math.log(2.0)))
    t = np.exp(-0.5 * ((xx / (0.1 * k)) ** 2 + (yy / (0.8 * k)) ** 2)) + 1e-4 * (xx * xx + yy * yy <= 4.0)
    t[t < 1e-30] = 0.0
    return t.astype(np.float32)


def _pattern(c, seed):
    r, rng = _raster(c), np.random.default_rng(seed + 17)
    na, ne = c["n_az"], c["n_el"]
    az = r.az_min + (np.arange(na) + 0.5) * (c["fov_az"] / na)
    el = r.el_min + (np.arange(ne) + 0.5) * (c["fov_el"] / ne)
    if c["steer"] == "lissajous":
        t = np.arange(na) / na
        p = int(rng.integers(50, 120))
        az = 0.475 * c["fov_az"] * np.sin(2.0 * math.pi * p * t + 0.5 * math.pi)
        el = 0.475 * c["fov_el"] * np.sin(2.0 * math.pi * (p - 1) * t)
    else:
        ee, aa = np.meshgrid(el, az, indexing="ij")
        az, el = aa.ravel(), ee.ravel()
        if c["steer"] == "jitter":
            az = az + rng.uniform(-0.5, 0.5, az.shape) * (c["fov_az"] / na)
            el = el + rng.uniform(-0.5, 0.5, el.shape) * (c["fov_el"] / ne)
    if c["pattern"] == "table":
        return SimpleNamespace(kind=lidar.LIDAR_PATTERN_TABLE, beam_az=az, beam_el=el, table=_table(), half_deg=(2.0, 2.0))
    return SimpleNamespace(kind=lidar.LIDAR_PATTERN_GAUSS, beam_az=az, beam_el=el,
                           sigma_deg=(c["sigma_az"], c["sigma_el"]), trunc_sigmas=3.0)


def _params(c):
    """Receiver: the scanning sensor's threshold (with its sun for the tabulated pattern), or the small sensor's."""
    small = c["bins"] == 512
    table = c.get("pattern") == "table"
    ambient = 1e-7 if small else 0.0 if table else 1e-8
    e, a = math.radians(30.0), math.radians(45.0)
    return SimpleNamespace(n_bins=c["bins"], bin_ns=c["bin_ns"], max_echoes=3,
                           threshold=ambient + 5e-6 if small else ROAD_THRESHOLD, emit_power=1.0, pulse_fwhm_ns=4.0,
                           pulse_trunc_sigmas=4.0, ambient_const=ambient, sun_irradiance=ROAD_SUN if table else 0.0,
                           sun_dir=(math.cos(e) * math.cos(a), math.cos(e) * math.sin(a), math.sin(e)),
                           echo_select=SELECT[c.get("select", "all")], range_mode=RANGES[c.get("range", "centre")])


def _frames(c, seed):
    """The frames of a batch, each a frame case: one sensor repeated, or a mix of sizes, scenes and footprints."""
    out = []
    for i in range(c["frames"]):
        f = dict(c, kind="frame")
        if c["mixed"]:
            k = i % 3
            f["scene"] = ("iid", "road")[i % 2]
            f["steer"] = ("grid", "lissajous", "jitter")[k]
            f["width"], f["height"] = max(64, c["width"] >> k) - k, max(32, c["height"] >> k)
            na, ne = max(4, c["n_az"] * (3 - k) // 3), max(4, c["n_el"] * (3 - k) // 3)
            f["n_az"], f["n_el"] = (na * ne, 1) if f["steer"] == "lissajous" else (na, ne)
            # 20 to 20000 pixels; the wide footprints on the small rasters' fewer beams
            s = math.sqrt((20.0, 150.0, 1000.0, 6000.0, 60.0, 20000.0)[i % 6] / math.pi) / 3.0
            f["sigma_az"], f["sigma_el"] = s * f["fov_az"] / f["width"], s * f["fov_el"] / f["height"]
        out.append((f, seed + 101 * i))
    return out


def _outputs(n, echoes=3):
    """Device buffers for a frame's echoes, counts and beam records, and typed views of their fields."""
    raw = torch.zeros((n, echoes * 40), dtype=torch.uint8, device="cuda")
    cnt = torch.zeros(n, dtype=torch.int32, device="cuda")
    beams = torch.zeros((n, 24), dtype=torch.uint8, device="cuda")
    f8, f4, i4 = (raw.view(t).view(n, echoes, -1) for t in (torch.float64, torch.float32, torch.int32))
    b4, bi = beams.view(torch.float32), beams.view(torch.int32)
    return raw, cnt, beams, {"range_m": f8[..., 0], "time_ns": f8[..., 1], "intensity": f4[..., 4],
                             "width_ns": f4[..., 5], "bins": i4[..., 6:10], "n_echoes": cnt, "pixel": bi[:, 0:2],
                             "scale": b4[:, 2], "floor": b4[:, 3], "samples": bi[:, 4]}


def _weights(seed):
    rng = np.random.default_rng(seed)
    parts = []
    for k, (i, o) in enumerate(SUR_LAYERS):
        used = 1030 if k == 0 else i
        w = rng.uniform(-1.0, 1.0, (i, o)) * math.sqrt(3.0 / used)
        w[used:] = 0.0
        if k == 3:
            w[:, 13:] = 0.0
        parts += [w.ravel(), rng.uniform(-0.1, 0.1, o)]
    return np.concatenate(parts).astype(np.float32)


def _rows(n, seed):
    """Network inputs (bfloat16 bits) in the ranges of the real channels, and labels."""
    g = torch.Generator("cuda").manual_seed(seed)
    x = torch.randn((n, 1056), generator=g, device="cuda") * 0.5
    x[:, 256:].clamp_(0.0, 1.0)
    x[:, 1030:] = 0.0
    lab = torch.zeros((n, 16), device="cuda")
    lab[:, :3] = (torch.rand((n, 3), generator=g, device="cuda") < 0.5).float()
    lab[:, 3:12] = torch.randn((n, 9), generator=g, device="cuda") * 0.5 * lab[:, :3].repeat(1, 3)
    return x.to(torch.bfloat16).view(torch.int16), lab


def prepare(case, seed):
    c, s = case, SimpleNamespace(case=case)
    stream = torch.cuda.current_stream()
    kind = c["kind"]
    if kind in ("forward", "gradients"):
        sim = lidar.LidarSim(_params(FRAME), stream=stream)
        sim.set_weights(_weights(seed))
        s.sim, (s.x, s.lab) = sim, _rows(c["rows"], seed)
        s.y = torch.zeros((c["rows"], 16), device="cuda")
        s.grads, s.loss = torch.zeros(SUR_PARAMS, device="cuda"), torch.zeros(1, device="cuda")
        return s
    if kind == "batch":
        s.sim = lidar.LidarSim(_params(c), stream=stream)
        fr = _frames(c, seed)
        pats = [_pattern(f, sd) for f, sd in fr]
        s.planes = [_planes(f, _raster(f), sd) for f, sd in fr]
        s.batch = lidar.Batch([(_raster(f), p) for (f, _), p in zip(fr, s.planes)], pats)
        s.off = np.cumsum([0] + [len(p.beam_az) for p in pats]).tolist()
        s.out = _outputs(s.off[-1])              # one array for all frames
        s.sim.simulate_batch(s.batch)            # the first call sets the batch up and captures its graph
        return s
    s.raster, s.params = _raster(c), _params(c)
    if kind == "stack":
        x = np.arange(-c["M"], c["M"] + 1) * (c["fov_az"] / c["width"])
        y = np.arange(-c["N"], c["N"] + 1) * (c["fov_el"] / c["height"])
        s.H = (np.exp(-0.5 * (x / c["core_az"]) ** 2) + 1e-4).astype(np.float32)
        s.V = np.exp(-0.5 * (y / c["core_el"]) ** 2).astype(np.float32)
        om = math.radians(c["fov_az"] / c["width"]) * math.radians(c["fov_el"] / c["height"])
        s.rho_min = 0.05 * float(s.H.sum(dtype=np.float64) * s.V.sum(dtype=np.float64)) * om * 0.5 / (math.pi * 1e4)
        s.planes = _planes(dict(c, scene="road"), s.raster, seed)
        s.sim = lidar.LidarSim(s.params, stream=stream)
        s.near = torch.zeros((c["height"], c["width"]), dtype=torch.int32, device="cuda")
        s.xi = torch.zeros((c["height"], c["width"]), device="cuda")
        return s
    s.pattern = _pattern(c, seed)
    s.out = _outputs(len(s.pattern.beam_az))
    if kind == "pinhole":
        s.src, s.planes = _pinhole(c, seed)
    else:
        s.planes = _planes(c, s.raster, seed)
    if kind != "static":
        s.sim = lidar.LidarSim(s.params, stream=stream)
        s.sim.set_pattern(s.pattern)
        if kind == "surrogate":
            # untrained weights: a gate that sends about one beam in eight to the plain path, as a trained network's does
            s.sim.set_weights(_weights(seed))
            s.sim.set_gbuffer(s.raster, s.planes)
            n = len(s.pattern.beam_az)
            x, y = torch.zeros((n, 1056), dtype=torch.int16, device="cuda"), torch.zeros((n, 16), device="cuda")
            s.sim.surrogate_features(x)
            s.sim.surrogate_forward(x, y)
            s.sim.set_gate(float(torch.sigmoid(torch.quantile(y[:, 12].double(), 0.125))), math.inf)
    return s


def run(s):
    c = s.case
    kind = c["kind"]
    if kind == "forward":
        s.sim.surrogate_forward(s.x, s.y)
        return s.y
    if kind == "gradients":
        s.sim.surrogate_gradients(s.x, s.lab, s.grads, s.loss)
        return s.grads, s.loss
    if kind == "stack":
        s.sim.set_gbuffer(s.raster, s.planes)
        s.sim.range_stacking(s.H, s.V, s.rho_min, s.near, s.xi)
        return s.near, s.xi
    if kind == "batch":
        s.sim.simulate_batch(s.batch)
        read = lidar.load().lidar_sim_read_batch
        raw, cnt, beams, views = s.out
        at = raw.data_ptr(), cnt.data_ptr(), beams.data_ptr()
        for i, o in enumerate(s.off[:-1]):
            rc = read(s.sim._h, i, at[0] + 120 * o, at[1] + 4 * o, None, at[2] + 24 * o, 1)
            if rc != lidar.LIDAR_OK:
                raise RuntimeError(s.sim.last_error())
        return views
    raw, cnt, beams, views = s.out
    if kind == "static":
        lidar.simulate_static(s.params, s.pattern, s.raster, s.planes, raw, cnt, beams,
                              stream=torch.cuda.current_stream())
        return views
    if kind == "pinhole":
        s.sim.set_gbuffer_pinhole(s.src, s.planes, s.raster)
    else:
        s.sim.set_gbuffer(s.raster, s.planes)
    s.sim.simulate_frame(lidar.LIDAR_MODE_SURROGATE if kind == "surrogate" else lidar.LIDAR_MODE_PLAIN)
    s.sim.read_device(echoes=raw, n_echoes=cnt, beams=beams)
    return views


# ---- the work of a pass ------------------------------------------------------------------------------------------


def _kernel(c, pattern, r):
    """The pattern on the pixel-offset grid: K[n + N][m + M] in 64 bits (numpy), M, N."""
    dphi, de = (r.az_max - r.az_min) / r.width, (r.el_max - r.el_min) / r.height
    if pattern.kind == lidar.LIDAR_PATTERN_GAUSS:
        (sx, sy), t = pattern.sigma_deg, pattern.trunc_sigmas
        M, N = math.floor(t * sx / dphi), math.floor(t * sy / de)
        y, x = np.meshgrid(np.arange(-N, N + 1) * de, np.arange(-M, M + 1) * dphi, indexing="ij")
        q = (x / sx) ** 2 + (y / sy) ** 2
        return np.where(q > t * t, 0.0, np.exp(-0.5 * q)), M, N
    hx, hy = pattern.half_deg
    M, N = math.floor(hx / dphi), math.floor(hy / de)
    ny, nx = pattern.table.shape
    tab = np.zeros((ny + 2, nx + 2))
    tab[1:-1, 1:-1] = pattern.table
    fx = (np.arange(-M, M + 1) * dphi + hx) / (2.0 * hx / nx) - 0.5
    fy = (hy + np.arange(-N, N + 1) * de) / (2.0 * hy / ny) - 0.5
    ix, iy = np.floor(fx).astype(int), np.floor(fy).astype(int)
    tx, ty = (fx - ix)[None], (fy - iy)[:, None]
    at = lambda j, i: tab[np.ix_(np.clip(j + 1, 0, ny + 1), np.clip(i + 1, 0, nx + 1))]  # noqa: E731
    return (1 - ty) * ((1 - tx) * at(iy, ix) + tx * at(iy, ix + 1)) + \
        ty * ((1 - tx) * at(iy + 1, ix) + tx * at(iy + 1, ix + 1)), M, N


def _beam_pixels(pattern, r):
    dphi, de = (r.az_max - r.az_min) / r.width, (r.el_max - r.el_min) / r.height
    return (np.floor((pattern.beam_az - r.az_min) / dphi).astype(np.int64),
            np.floor((r.el_max - pattern.beam_el) / de).astype(np.int64))


def _frame_work(c, seed=0):
    """Planes read once, echoes, counts and beam records written; 6 operations a sample, 8 with the sun."""
    r, pattern = _raster(c), _pattern(c, seed)
    K, M, N = _kernel(c, pattern, r)
    box = np.zeros((K.shape[0] + 1, K.shape[1] + 1))
    box[1:, 1:] = (K > 0).cumsum(0).cumsum(1)
    u, v = _beam_pixels(pattern, r)
    c0, c1 = np.clip(M - u, 0, 2 * M + 1), np.clip(r.width - u + M, 0, 2 * M + 1)
    r0, r1 = np.clip(N - v, 0, 2 * N + 1), np.clip(r.height - v + N, 0, 2 * N + 1)
    samples = float((box[r1, c1] - box[r0, c1] - box[r1, c0] + box[r0, c0]).sum())
    per = 8.0 if c["pattern"] == "table" else 6.0
    return {"bytes": 24.0 * min(r.width * r.height, samples) + len(u) * (3 * 40 + 4 + 24), "flops": per * samples}


SUR_FLOPS = 2.0 * sum(i * o for i, o in SUR_LAYERS)


def work(case):
    c = case
    kind = c["kind"]
    if kind == "forward":
        return {"bytes": c["rows"] * (1056 * 2 + 64) + 2.0 * SUR_PARAMS, "flops": SUR_FLOPS * c["rows"]}
    if kind == "gradients":
        # forward, weight gradients, input gradients of all layers but the first
        back = SUR_FLOPS + 2.0 * sum(i * o for i, o in SUR_LAYERS[1:])
        return {"bytes": c["rows"] * (1056 * 2 + 64) + 6.0 * SUR_PARAMS, "flops": (SUR_FLOPS + back) * c["rows"]}
    if kind == "stack":
        # every pixel's value enters the slice sums of 2 N + 1 rows after one row sum each of 2 M + 1 columns
        px = float(c["width"] * c["height"])
        return {"bytes": px * (24 + 8), "flops": 2.0 * px * (2 * c["M"] + 1 + (2 * c["M"] + 1) * (2 * c["N"] + 1))}
    if kind == "batch":
        parts = [_frame_work(f, sd) for f, sd in _frames(c, 0)]
        return {k: sum(p[k] for p in parts) for k in ("bytes", "flops")}
    w = _frame_work(c)
    if kind == "pinhole":
        w["bytes"] += 24.0 * c["src_w"] * c["src_h"]
    if kind == "surrogate":
        b = c["n_az"] * c["n_el"]
        w = {"bytes": 24.0 * c["width"] * c["height"] + b * (3 * 40 + 4 + 24), "flops": SUR_FLOPS * b}
    return w


# ---- outputs in 64 bits ------------------------------------------------------------------------------------------


def _exact_pinhole_planes(c, src, planes):
    """The planes on the equiangular raster: nearest pinhole pixel, decoded range, turned normal (float32 as stored)."""
    r = _raster(c)
    d = _directions(r)
    rot = src.rot
    cam = [sum(float(rot[j, i]) * d[j] for j in range(3)) for i in range(3)]
    front = cam[2] > 0.0
    z = torch.where(front, cam[2], 1.0)
    i, j = torch.floor(src.fx * cam[0] / z + src.cx), torch.floor(src.fy * cam[1] / z + src.cy)
    ok = front & (i >= 0) & (i < src.width) & (j >= 0) & (j < src.height)
    i, j = torch.where(ok, i, 0.0), torch.where(ok, j, 0.0)
    at = j.long() * src.width + i.long()
    take = [p.reshape(-1)[at].double() for p in planes]
    w = take[0] / 16777215.0
    ok &= (w >= 0.0) & (w < 1.0)
    rx, ry = (i + 0.5 - src.cx) / src.fx, (j + 0.5 - src.cy) / src.fy
    dep = src.near * src.far / (src.far - w * (src.far - src.near)) * torch.sqrt(rx * rx + ry * ry + 1.0)
    n = [sum(float(rot[k, m]) * take[3 + m] for m in range(3)) for k in range(3)]
    sky = (math.inf, 0.0, 1.0, 0.0, 0.0, 0.0)
    return tuple(torch.where(ok, v, o).float() for v, o in zip((dep, take[1], take[2], *n), sky))


def _exact_frame(c, pattern, planes):
    r, p = _raster(c), _params(c)
    f64 = dict(dtype=torch.float64, device="cuda")
    dphi, de = (r.az_max - r.az_min) / r.width, (r.el_max - r.el_min) / r.height
    W, H, R = r.width, r.height, p.n_bins
    depth, rho, gain, nx, ny, nz = (t.double() for t in planes)
    d = _directions(r)
    edge = torch.sin(torch.deg2rad(r.el_max - torch.arange(H + 1, **f64) * de))
    omega = (math.radians(dphi) * (edge[:-1] - edge[1:]))[:, None]
    to_bin = 2.0 / (LIGHT * (p.bin_ns * 1e-9))
    ok = torch.isfinite(depth) & (depth > 0.0)
    depth = torch.where(ok, depth, 1.0)
    kb = torch.floor(depth * to_bin)
    ok &= kb < R
    bins = torch.where(ok, kb, 0.0).long().reshape(-1)
    cos = (-(nx * d[0] + ny * d[1] + nz * d[2])).clamp(min=0.0)
    shade = torch.where(ok, omega * gain * rho / math.pi * cos / depth ** 2, 0.0).reshape(-1)
    sd = p.sun_dir
    lit = (nx * sd[0] + ny * sd[1] + nz * sd[2]).clamp(min=0.0)
    sun = torch.where(ok, omega * rho / math.pi * lit, 0.0).reshape(-1)
    K, M, N = _kernel(c, pattern, r)
    K = torch.from_numpy(K).cuda()
    u, v = (torch.from_numpy(t).cuda() for t in _beam_pixels(pattern, r))
    B = len(u)
    # normalisation over the whole kernel (rows outside the image included)
    rows = v[:, None] + torch.arange(-N, N + 1, device="cuda")[None]
    row_om = math.radians(dphi) * (torch.sin(torch.deg2rad(r.el_max - rows.double() * de)) -
                                   torch.sin(torch.deg2rad(r.el_max - (rows.double() + 1.0) * de)))
    scale = p.emit_power / (row_om * K.sum(1)[None]).sum(1)
    xi, e_sun = torch.zeros((B, R), **f64), torch.zeros(B, **f64)
    corrected = p.range_mode == lidar.LIDAR_RANGE_CORRECTED
    cols = torch.arange(-M, M + 1, device="cuda")
    step = max(1, int(2.4e7 // K.numel()))
    if corrected:
        az, el = _angles(r)
        beam_az, beam_el = (torch.from_numpy(np.asarray(t)).cuda() for t in (pattern.beam_az, pattern.beam_el))
        pn = nx * d[0] + ny * d[1] + nz * d[2]
    for b0 in range(0, B, step):
        vv, uu = rows[b0:b0 + step, :, None], (u[b0:b0 + step, None] + cols[None])[:, None, :]
        nb = len(vv)
        inside = (vv >= 0) & (vv < H) & (uu >= 0) & (uu < W) & (K > 0.0)[None]
        beam, kr, kc = torch.nonzero(inside, as_tuple=True)
        px = (v[b0 + beam] + kr - N) * W + (u[b0 + beam] + kc - M)
        kv = K[kr, kc]
        k, wgt = bins[px], kv * shade[px]
        if corrected:
            # the range on the pixel's plane along the kernel cell's own direction
            a = torch.deg2rad(beam_az[b0 + beam] + (kc - M) * dphi)
            e = torch.deg2rad(beam_el[b0 + beam] - (kr - N) * de)
            ce = torch.cos(e)
            vn = ce * torch.cos(a) * nx.reshape(-1)[px] + ce * torch.sin(a) * ny.reshape(-1)[px] + torch.sin(e) * nz.reshape(-1)[px]
            q = pn.reshape(-1)[px] / vn
            q = torch.where(q > 0.0, q, 2.0).clamp(0.5, 2.0)
            k = torch.floor(depth.reshape(-1)[px] * q * to_bin).long()
            wgt = torch.where(k < R, wgt, 0.0)
            k = k.clamp(max=R - 1)
        xi[b0:b0 + nb].view(-1).index_add_(0, beam * R + k, wgt)
        if p.sun_irradiance:
            e_sun[b0:b0 + nb].index_add_(0, beam, kv * sun[px])
    floor = p.ambient_const + p.sun_irradiance / float(K.max()) * e_sun
    xi *= scale[:, None]
    T = p.threshold
    out = {"pixel": None, "bins": None, "samples": None, "n_echoes": None, "scale": scale, "floor": floor}
    idx = torch.arange(R, device="cuda")[None]
    E = p.max_echoes
    res = {k: torch.zeros((B, E), **f64) for k in ("range_m", "time_ns", "intensity", "width_ns")}

    def put(e, has, peak, best, width):
        res["range_m"][:, e] = torch.where(has, 0.5 * LIGHT * p.bin_ns * 1e-9 * (peak + 0.5), 0.0)
        res["time_ns"][:, e] = torch.where(has, p.bin_ns * (peak + 0.5), 0.0)
        res["intensity"][:, e] = torch.where(has, best, 0.0)
        res["width_ns"][:, e] = torch.where(has, width, 0.0)
    if p.echo_select == lidar.LIDAR_ECHO_RAW_NEAREST:
        hit = xi >= T
        has, peak = hit.any(1), torch.where(hit, idx, R).amin(1).clamp(max=R - 1)
        put(0, has, peak, xi.gather(1, peak[:, None])[:, 0], torch.zeros(B, **f64))
        return {**out, **res}
    sigma = p.pulse_fwhm_ns / (2.0 * math.sqrt(2.0 * math.log(2.0)))
    J = math.ceil(p.pulse_trunc_sigmas * sigma / p.bin_ns)
    taps = np.exp(-0.5 * (np.arange(-J, J + 1) * p.bin_ns / sigma) ** 2)
    taps /= taps.sum()
    pad = torch.nn.functional.pad(xi, (J, J))
    xh = floor[:, None].expand(B, R).clone()
    for j in range(2 * J + 1):
        xh += float(taps[j]) * pad[:, 2 * J - j:2 * J - j + R]
    above = xh > T
    below = torch.nn.functional.pad(above, (1, 1)) == 0                       # bins -1 .. R
    at = torch.arange(-1, R + 1, device="cuda")[None].expand(B, R + 2)
    prev = torch.where(below, at, -1).cummax(1).values[:, 1:-1]               # last bin below, at or before
    nxt = torch.where(below, at, R).flip(1).cummin(1).values.flip(1)[:, 1:-1]
    runs = (above & (prev == idx - 1)).cumsum(1)
    for e in range(E if p.echo_select == lidar.LIDAR_ECHO_ALL else 1):
        mine = above if p.echo_select == lidar.LIDAR_ECHO_STRONGEST else above & (runs == e + 1)
        has = mine.any(1)
        best = torch.where(mine, xh, -math.inf).amax(1)
        peak = torch.where(mine & (xh == best[:, None]), idx, R).amin(1).clamp(max=R - 1)
        k0 = prev.gather(1, peak[:, None])[:, 0] + 1
        k1 = nxt.gather(1, peak[:, None])[:, 0] - 1

        def val(k):
            return xh.gather(1, k.clamp(0, R - 1)[:, None])[:, 0]
        up = torch.where(k0 == 0, 0.5, (T - val(k0 - 1)) / (val(k0) - val(k0 - 1)))
        dn = torch.where(k1 == R - 1, 0.5, (val(k1) - T) / (val(k1) - val(k1 + 1)))
        put(e, has, peak, best - floor, (k1 - k0 + 1 + dn - up) * p.bin_ns)
    return {**out, **res}


def _exact_mlp(seed, x):
    w, o, layers = torch.from_numpy(_weights(seed)).cuda().double(), 0, []
    w.requires_grad_(True)
    for i, n in SUR_LAYERS:
        layers.append((w[o:o + i * n].view(i, n), w[o + i * n:o + i * n + n]))
        o += i * n + n
    h = x.view(torch.bfloat16).double()
    for k, (a, b) in enumerate(layers):
        h = h @ a + b
        if k < 3:
            h = torch.nn.functional.gelu(h)
    return w, h


def exact(case, seed):
    c = case
    kind = c["kind"]
    if kind == "surrogate":
        return None                               # gate decisions select between two methods
    if kind in ("forward", "gradients"):
        x, lab = _rows(c["rows"], seed)
        if kind == "forward":
            with torch.no_grad():
                return _exact_mlp(seed, x)[1]
        w, y = _exact_mlp(seed, x)
        lab = lab.double()
        ex, bce = lab[:, :3], torch.nn.functional.binary_cross_entropy_with_logits
        bad = ((y[:, :3] > 0) != (ex > 0.5)) | ((ex > 0.5) & (((y[:, 3:6] - lab[:, 3:6]).abs() * 16.0 > 0.5) |
                                                              (lab[:, 3:6].abs() >= 4.0)))
        sq = (y[:, 3:12] - lab[:, 3:12]) ** 2
        per = 64.0 * sq[:, 0:3] + sq[:, 3:6] + sq[:, 6:9]
        loss = (bce(y[:, :3], ex, reduction="none") + ex * per).sum(1).mean() + \
            bce(y[:, 12], (~bad.any(1)).double(), reduction="mean")
        loss.backward()
        return w.grad, loss.detach().view(1)
    if kind == "batch":
        parts = [_exact_frame(f, _pattern(f, sd), _planes(f, _raster(f), sd)) for f, sd in _frames(c, seed)]
        return {k: None if v is None else torch.cat([q[k] for q in parts]) for k, v in parts[0].items()}
    if kind == "stack":
        s = prepare(case, seed)
        r = s.raster
        depth, rho, gain, nx, ny, nz = (t.double() for t in s.planes)
        d = _directions(r)
        f64 = dict(dtype=torch.float64, device="cuda")
        edge = torch.sin(torch.deg2rad(r.el_max - torch.arange(r.height + 1, **f64) * (c["fov_el"] / r.height)))
        omega = (math.radians(c["fov_az"] / r.width) * (edge[:-1] - edge[1:]))[:, None]
        k = torch.floor(torch.where(torch.isfinite(depth), depth, -1.0) * (2.0 / (LIGHT * (c["bin_ns"] * 1e-9))))
        cos = (-(nx * d[0] + ny * d[1] + nz * d[2])).clamp(min=0.0)
        shade = omega * gain * rho / math.pi * cos / depth ** 2
        xi, found = torch.zeros_like(shade), torch.zeros_like(shade, dtype=torch.bool)
        fits = (k >= 0) & (k < c["bins"])
        for sl in torch.unique(k[fits]).tolist():
            img = torch.where(k == sl, shade, 0.0)
            for dim, taps in ((1, s.H), (0, s.V)):
                half = len(taps) // 2
                pad = torch.nn.functional.pad(img, (half, half) if dim == 1 else (0, 0, half, half))
                n = img.shape[dim]
                img = torch.zeros_like(img)
                for j, t in enumerate(taps):
                    img.add_(pad.narrow(dim, j, n), alpha=float(t))
            hit = (img >= s.rho_min) & ~found
            xi, found = torch.where(hit, img, xi), found | hit
        return None, xi
    pattern = _pattern(c, seed)
    if kind == "pinhole":
        return _exact_frame(c, pattern, _exact_pinhole_planes(c, *_pinhole(c, seed)))
    return _exact_frame(c, pattern, _planes(c, _raster(c), seed))

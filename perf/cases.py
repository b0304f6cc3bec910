"""The work that users of this framework have it do, as measurable cases.

Scenes are multi-scan indoor LiDAR clouds (scanners casting rays uniform on the
sphere into walls with doors, boxes and spheres; colour noise, per-scan gains
and occlusion gaps), networks He-initialised U-Nets: the workloads of
``synth/`` made on the GPU, so that new inputs are quick to make.  Geometry
results (key, depth, rgba) are selections among the cloud's points, defined
bit for bit; U-Net outputs have a float64 value.
"""

import math
import struct

import numpy as np
import torch

import paper_2502_11618_amd as L

PRECISIONS = {"fp32": L.LNR_FP32, "fp16": L.LNR_FP16, "bf16": L.LNR_BF16, "bf16x3": L.LNR_BF16X3,
              "fp8": L.LNR_FP8_E4M3, "fp8x3": L.LNR_FP8_E4M3X3}


def listed():
    return [
        # one small preview frame, start to end: the smallest calls, where launches and latency count
        dict(name="frame-room-256-fp32", kind="frame", points=200_000, rooms=1, cell=0.5, width=256, height=256,
             fov=70.0, levels=4, strength=0.5, precision="fp32", widths="16,32,64"),
        # the usual frame: a 20M-point scan at 1080p, projected, filtered and reconstructed at 16 bits
        dict(name="frame-20m-1080p-fp16", kind="frame", points=20_000_000, rooms=8, cell=1.0, width=1920, height=1080,
             fov=90.0, levels=5, strength=0.5, precision="fp16", widths="32,64,128,256"),
        # projection and depth filter alone (an unreconstructed viewer): a large scan at 1440p
        dict(name="project-100m-1440p", kind="project", points=100_000_000, rooms=8, cell=1.0, width=2560, height=1440,
             fov=90.0, levels=5, strength=0.5),
        # the soft z-buffer, at an odd window size
        dict(name="soft-5m-1003x747", kind="soft", points=5_000_000, rooms=8, cell=1.0, width=1003, height=747,
             fov=80.0, levels=4, strength=0.5, eps=0.01),
        # the views of several viewers projected in one call
        dict(name="views-8x1080p-20m", kind="views", points=20_000_000, rooms=8, cell=1.0, width=1920, height=1080,
             fov=90.0, views=8),
        # reconstruction of one 1080p image in float32 (the default precision)
        dict(name="unet-fp32-1080p", kind="unet", width=1920, height=1080, precision="fp32", widths="32,64,128,256"),
        # the largest reconstruction: 4K, five levels, 16 bits
        dict(name="unet-fp16-4k", kind="unet", width=3840, height=2160, precision="fp16", widths="32,64,128,256,512"),
        # split bfloat16 (float32-like accuracy) at the smaller window size
        dict(name="unet-bf16x3-960x720", kind="unet", width=960, height=720, precision="bf16x3",
             widths="32,64,128,256"),
        # split e4m3 at 1440p
        dict(name="unet-fp8x3-1440p", kind="unet", width=2560, height=1440, precision="fp8x3",
             widths="32,64,128,256"),
        # bfloat16 on a window that no tile divides, with widths that are no powers of two
        dict(name="unet-bf16-1284x724", kind="unet", width=1284, height=724, precision="bf16", widths="48,96,192"),
        # a serving step: eight sessions' cameras submitted, batched, rendered and reconstructed
        dict(name="serve-8x720p-fp16", kind="serve", points=20_000_000, rooms=8, cell=1.0, width=1280, height=720,
             fov=90.0, levels=5, strength=0.5, precision="fp16", widths="32,64,128,256", sessions=8),
        # loading a scan from host memory (partition, sort, boxes), once per cloud
        dict(name="load-5m", kind="load", points=5_000_000, rooms=8, cell=1.0),
    ]


def draw(rng):
    def logint(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    def size(lo, hi, multiple):
        w = max(multiple, logint(lo, hi) // multiple * multiple)
        h = max(multiple, int(w * rng.choice([0.5625, 0.75, 1.0])) // multiple * multiple)
        return w, h

    kind = rng.choice(["frame", "project", "soft", "views", "unet", "unet", "unet", "serve", "load"])
    if kind == "load":
        return dict(kind=kind, points=logint(10_000, 20_000_000), rooms=rng.choice([1, 8]),
                    cell=rng.choice([0.5, 1.0, 2.0]))
    case = dict(kind=kind)
    multiple = 1
    if kind in ("frame", "unet", "serve"):
        n = rng.choice([3, 3, 4, 4, 5]) if kind == "unet" else rng.choice([3, 4])
        base = rng.choice([16, 32, 32, 48])
        case["widths"] = ",".join(str(min(512, base << l)) for l in range(n))
        case["precision"] = rng.choice(sorted(PRECISIONS))
        multiple = 1 << (n - 1)
    if kind == "unet":
        while True:
            case["width"], case["height"] = size(160, 3840, multiple)
            f = _unet_flops(case)
            if f <= (7e11 if case["precision"] in ("fp32", "bf16x3", "fp8x3") else 3.2e12):
                return case
    few = kind in ("frame", "serve")
    case["points"] = logint(100_000, 20_000_000)
    case["rooms"] = 1 if case["points"] < 1_000_000 else 8
    case["cell"] = 0.5 if case["rooms"] == 1 else rng.choice([1.0, 2.0])
    case["width"], case["height"] = size(160, 1280 if few or kind == "views" else 2560, multiple)
    case["fov"] = rng.choice([60.0, 75.0, 90.0])
    if kind == "views":
        case["views"] = rng.choice([2, 3, 8, 11])
        return case
    case["levels"] = rng.choice([3, 4, 5, 6])
    case["strength"] = rng.choice([0.25, 0.5, 1.0])
    if kind == "soft":
        case["eps"] = rng.choice([0.005, 0.01, 0.05])
    if kind == "serve":
        case["sessions"] = rng.choice([1, 3, 8])
    return case


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

class _Camera:
    z_near, z_far = 0.1, 1000.0

    def __init__(self, eye, yaw, pitch, width, height, fov):
        fwd = np.array([math.cos(pitch) * math.cos(yaw), math.cos(pitch) * math.sin(yaw), math.sin(pitch)])
        right = np.cross(fwd, [0.0, 0.0, 1.0])
        right /= np.linalg.norm(right)
        R = np.stack([right, np.cross(fwd, right), fwd])
        f = (width / 2.0) / math.tan(math.radians(fov) / 2.0)
        K = np.array([[f, 0.0, width / 2.0], [0.0, f, height / 2.0], [0.0, 0.0, 1.0]])
        self.P = (K @ np.concatenate([R, (-R @ eye)[:, None]], axis=1)).astype(np.float32).reshape(12)
        self.width, self.height = width, height
        self.eye, self.R, self.f = eye, R, f


class _Scene:
    """Walls with doors, boxes and spheres; rooms of 10 x 15 x 6 m, or one of 10 x 8 x 3 m."""

    def __init__(self, seed, rooms):
        rng = np.random.default_rng([seed, 5])
        single = rooms == 1
        nx, ny = (1, 1) if single else (4, 2)
        rw, rd, Z = (10.0, 8.0, 3.0) if single else (10.0, 15.0, 6.0)
        X, Y = nx * rw, ny * rd
        rects = [(0, 0.0, 0, Y, 0, Z), (0, X, 0, Y, 0, Z), (1, 0.0, 0, X, 0, Z), (1, Y, 0, X, 0, Z),
                 (2, 0.0, 0, X, 0, Y), (2, Z, 0, X, 0, Y)]
        for i in range(1, nx):
            for j in range(ny):
                d = rng.uniform(j * rd + 0.5, (j + 1) * rd - 1.7)
                rects += [(0, i * rw, j * rd, d, 0, Z), (0, i * rw, d + 1.2, (j + 1) * rd, 0, Z),
                          (0, i * rw, d, d + 1.2, 2.2, Z)]
        for j in range(1, ny):
            for i in range(nx):
                d = rng.uniform(i * rw + 0.5, (i + 1) * rw - 1.7)
                rects += [(1, j * rd, i * rw, d, 0, Z), (1, j * rd, d + 1.2, (i + 1) * rw, 0, Z),
                          (1, j * rd, d, d + 1.2, 2.2, Z)]
        self.rects = rects
        self.centers = [np.array([(i + 0.5) * rw, (j + 0.5) * rd, 1.6]) for j in range(ny) for i in range(nx)]
        self.boxes, self.spheres = [], []
        clear = 1.4 if single else 3.6  # room centres stay free for scanners and cameras
        while len(self.boxes) < (0 if single else 32):
            s = rng.uniform([0.3, 0.3, 0.3], [2.0, 2.0, 2.5])
            lo = np.array([rng.uniform(0.2, X - s[0] - 0.2), rng.uniform(0.2, Y - s[1] - 0.2), 0.0])
            if min(np.hypot(*(lo[:2] + s[:2] / 2 - c[:2])) for c in self.centers) > clear + 1.0:
                self.boxes.append((lo, lo + s))
        while len(self.spheres) < (14 if single else 8):
            r = rng.uniform(0.2, 0.9)
            c = rng.uniform([r, r, r], [X - r, Y - r, Z - r])
            if min(np.hypot(*(c[:2] - k[:2])) for k in self.centers) > clear + r:
                self.spheres.append((c, r))
        n = len(rects) + len(self.boxes) + len(self.spheres)
        self.colors = torch.tensor(rng.integers(30, 226, size=(n, 3)), dtype=torch.float32, device="cuda")
        self.rng = rng
        self.reach = 1.0 if single else 3.0

    def cast(self, eye, d):
        """Nearest hit distance and surface along unit directions d [n, 3] from eye."""
        o = [float(v) for v in eye]
        t_best = torch.full((d.shape[0],), 1e9, device="cuda")
        sid = torch.zeros(d.shape[0], dtype=torch.int64, device="cuda")
        inv = 1.0 / torch.where(d.abs() < 1e-9, torch.full_like(d, 1e-9), d)

        def take(k, t, ok):
            ok = ok & (t > 0.05) & (t < t_best)
            t_best.copy_(torch.where(ok, t, t_best))
            sid.masked_fill_(ok, k)

        k = 0
        for axis, c, lo1, hi1, lo2, hi2 in self.rects:
            a1, a2 = [a for a in range(3) if a != axis]
            t = (c - o[axis]) * inv[:, axis]
            p1, p2 = o[a1] + t * d[:, a1], o[a2] + t * d[:, a2]
            take(k, t, (p1 >= lo1) & (p1 <= hi1) & (p2 >= lo2) & (p2 <= hi2))
            k += 1
        for lo, hi in self.boxes:
            e = torch.tensor(eye, dtype=torch.float32, device="cuda")
            t1 = (torch.tensor(lo, dtype=torch.float32, device="cuda") - e) * inv
            t2 = (torch.tensor(hi, dtype=torch.float32, device="cuda") - e) * inv
            tn, tf = torch.minimum(t1, t2).amax(1), torch.maximum(t1, t2).amin(1)
            take(k, tn, tn <= tf)
            k += 1
        for c, r in self.spheres:
            oc = torch.tensor(np.asarray(eye) - c, dtype=torch.float32, device="cuda")
            b = d @ oc
            disc = b * b - float(oc @ oc) + r * r
            take(k, -b - disc.clamp(min=0).sqrt(), disc >= 0)
            k += 1
        return t_best, sid

    def scan(self, g, n, scans):
        """n points of `scans` scanners, host arrays xyz float32 [n, 3] and rgb uint8 [n, 3]."""
        xyz, rgb = np.empty((n, 3), np.float32), np.empty((n, 3), np.uint8)
        at = 0
        for k in range(scans):
            eye = self.centers[k % len(self.centers)] + self.rng.uniform([-1, -1, -0.2], [1, 1, 0.0])
            gain = torch.tensor(self.rng.normal(1.0, 0.05, 3), dtype=torch.float32, device="cuda")
            gaps = self.rng.normal(size=(5 if scans > 1 else 0, 3))
            end = n * (k + 1) // scans
            while at < end:
                m = min(8_000_000, int((end - at) * 1.15) + 4096)
                z = torch.rand(m, device="cuda", generator=g) * 2 - 1
                phi = torch.rand(m, device="cuda", generator=g) * (2 * math.pi)
                xy = (1 - z * z).sqrt()
                d = torch.stack([xy * phi.cos(), xy * phi.sin(), z], 1)
                for c in gaps:
                    c = torch.tensor(c / np.linalg.norm(c), dtype=torch.float32, device="cuda")
                    d = d[d @ c < 0.97]
                d = d[:end - at]
                t, sid = self.cast(eye, d)
                p = torch.tensor(eye, dtype=torch.float32, device="cuda") + t[:, None] * d
                c = self.colors[sid] + 8.0 * torch.randn(d.shape, device="cuda", generator=g)
                c = (c * gain).round().clamp(0, 255).to(torch.uint8)
                xyz[at:at + len(d)], rgb[at:at + len(d)] = p.cpu().numpy(), c.cpu().numpy()
                at += len(d)
        return xyz, rgb

    def camera(self, width, height, fov):
        th = self.rng.uniform(0, 2 * math.pi)
        eye = self.centers[0] + self.reach * np.array([math.cos(th), math.sin(th), 0.0])
        return _Camera(eye, th + math.pi + math.radians(20), math.radians(-10), width, height, fov)


def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _scan(case, seed):
    scene = _Scene(seed, case["rooms"])
    xyz, rgb = scene.scan(_generator(seed), case["points"], 1 if case["rooms"] == 1 else 4)
    return scene, xyz, rgb


def _layers(widths):
    w, out = widths, []
    for l in range(len(w)):
        out += [(w[l], 5 if l == 0 else w[l - 1], 3), (w[l], w[l], 3)]
    for l in range(len(w) - 2, -1, -1):
        out += [(w[l], w[l] + w[l + 1], 3), (w[l], w[l], 3)]
    return out + [(3, w[0], 1)]


def _widths(case):
    return [int(x) for x in case["widths"].split(",")]


def _weights(widths, seed):
    """He-normal weights and small biases of every convolution, in blob order."""
    rng = np.random.default_rng([seed, 42])
    return [(rng.standard_normal((co, ci, k, k), dtype=np.float32) * np.float32(math.sqrt(2.0 / (ci * k * k))),
             rng.uniform(-0.1, 0.1, co).astype(np.float32)) for co, ci, k in _layers(widths)]


def _net(ctx, case, seed):
    widths = _widths(case)
    parts = [b"LNRU", struct.pack("<4I", 1, len(widths), 5, 3), struct.pack(f"<{len(widths)}I", *widths)]
    for w, b in _weights(widths, seed):
        parts += [struct.pack("<3I", *w.shape[:3]), w.tobytes(), b.tobytes()]
    return L.lnr_unet_load(ctx, b"".join(parts), PRECISIONS[case["precision"]])


def _picture(case, seed):
    """An RGBDA image as a filtered projection leaves it: surfaces with about a third of the pixels empty."""
    W, H = case["width"], case["height"]
    scene, g = _Scene(seed, 8), _generator(seed)
    cam = scene.camera(W, H, 90.0)
    y, x = torch.meshgrid(torch.arange(H, device="cuda") + 0.5, torch.arange(W, device="cuda") + 0.5, indexing="ij")
    local = torch.stack([(x - W / 2) / cam.f, (y - H / 2) / cam.f, torch.ones_like(x)], -1).reshape(-1, 3)
    norm = local.norm(dim=1, keepdim=True)
    t, sid = scene.cast(cam.eye, (local / norm) @ torch.tensor(cam.R, dtype=torch.float32, device="cuda"))
    fill = torch.rand(t.shape, device="cuda", generator=g) < 0.65
    depth = torch.where(fill, t / norm[:, 0], torch.zeros_like(t))
    c = scene.colors[sid] + 8.0 * torch.randn(local.shape, device="cuda", generator=g)
    rgba = torch.cat([c.round().clamp(0, 255), torch.ones_like(t)[:, None]], 1) * fill[:, None]
    return depth.reshape(H, W).contiguous(), rgba.to(torch.uint8).reshape(H, W, 4).contiguous()


# ---------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------

def prepare(case, seed):
    kind = case["kind"]
    s = dict(case=case, ctx=L.lnr_context_create(0))
    if kind == "unet":
        s["net"] = _net(s["ctx"], case, seed)
        s["image"] = L.Image.from_tensors(*_picture(case, seed))
        s["rgb"] = torch.empty((3, case["height"], case["width"]), device="cuda")
        return s
    scene, xyz, rgb = _scan(case, seed)
    if kind == "load":
        s["xyz"], s["colors"] = xyz, rgb
        return s
    s["cloud"] = L.lnr_cloud_load(s["ctx"], xyz, rgb, case["cell"])
    W, H = case["width"], case["height"]
    n = case.get("views", case.get("sessions", 1))
    s["cams"] = [L.lnr_camera(*_plain(scene.camera(W, H, case["fov"]))) for _ in range(n)]
    if kind in ("frame", "serve"):
        s["net"] = _net(s["ctx"], case, seed)
    if kind == "serve":
        s["server"] = L.lnr_server_create(s["ctx"], s["cloud"], s["net"], max_batch=8, lanes=2,
                                          n_levels=case["levels"], filter_strength=case["strength"], max_width=W,
                                          max_height=H)
        s["sessions"] = [L.lnr_server_open_session(s["server"], W, H) for _ in range(n)]
        s["rgb"] = [torch.empty((3, H, W), device="cuda") for _ in range(n)]
        return s
    s["images"] = [L.Image(H, W) for _ in range(n)]
    s["rgb"] = torch.empty((3, H, W), device="cuda")
    return s


def _plain(cam):
    import ctypes
    return (ctypes.c_float * 12)(*[float(v) for v in cam.P]), cam.width, cam.height, cam.z_near, cam.z_far


def run(s):
    case, ctx = s["case"], s["ctx"]
    kind = case["kind"]
    if kind == "unet":
        L.lnr_reconstruct(ctx, s["net"], s["image"], s["rgb"])
        return s["rgb"]
    if kind == "load":
        cloud = L.lnr_cloud_load(ctx, s["xyz"], s["colors"], case["cell"])
        return L.lnr_cloud_permutation(cloud).view(np.int32), L.lnr_cloud_cell_start(cloud).view(np.int32)
    if kind == "serve":
        srv = s["server"]
        for k, (sid, cam) in enumerate(zip(s["sessions"], s["cams"])):
            L.lnr_server_submit(srv, sid, cam, k)
        left = len(s["sessions"])
        while left:
            L.lnr_server_step(srv)
            for r in L.lnr_server_poll(srv, 16):
                L.copy_from_device(r["rgb"], s["rgb"][r["tag"]])
                left -= 1
        return s["rgb"]
    if kind == "views":
        L.lnr_render_views(ctx, s["cloud"], s["cams"], s["images"])
        return [(i.key, i.depth, i.rgba) for i in s["images"]]
    img = s["images"][0]
    if kind == "soft":
        L.lnr_render_soft(ctx, s["cloud"], s["cams"][0], img, case["eps"])
    else:
        L.lnr_render(ctx, s["cloud"], s["cams"][0], img)
    L.lnr_depth_filter(ctx, img, case["levels"], case["strength"])
    if kind == "frame":
        L.lnr_reconstruct(ctx, s["net"], img, s["rgb"])
        return img.key, img.depth, img.rgba, s["rgb"]
    return img.key, img.depth, img.rgba


def _unet_flops(case):
    w, px, f = _widths(case), case["width"] * case["height"], 0
    shapes = _layers(w)
    levels = [l for l in range(len(w)) for _ in (0, 1)] + [l for l in range(len(w) - 2, -1, -1) for _ in (0, 1)] + [0]
    for (co, ci, k), l in zip(shapes, levels):
        f += 2 * co * ci * k * k * (px >> (2 * l))
    return f


def work(case):
    """Projection reads the points in view (about the share of the scene in front of the camera, 12 bytes each)
    and writes 16 bytes a pixel; the filter reads and writes depth and colour; the U-Net reads the image and its
    weights and writes the picture."""
    kind = case["kind"]
    if kind == "load":
        return {"bytes": case["points"] * (15 + 16 + 4), "flops": 0}
    px = case["width"] * case["height"]
    n = case.get("views", case.get("sessions", 1))
    b = f = 0
    if kind != "unet":
        # one or two of the eight rooms in view; the points of several views are read once
        b += case["points"] * (0.3 if case["rooms"] == 8 else 0.6) * (16 if kind == "soft" else 12)
        b += n * px * 16
        if "levels" in case:
            b += n * px * 8
    if "widths" in case:
        f = n * _unet_flops(case)
        size = 4 if case["precision"] in ("fp32", "bf16x3") else 2
        b += n * px * (8 + 12) + sum(co * ci * k * k for co, ci, k in _layers(_widths(case))) * size
    return {"bytes": b, "flops": f}


def _conv64(x, w, b):
    """x [C, H, W] float64, zero padding; one matrix product per tap."""
    co, _, k, _ = w.shape
    C, H, W = x.shape
    w = torch.tensor(w, device="cuda", dtype=torch.float64)
    y = torch.tensor(b, device="cuda", dtype=torch.float64)[:, None].expand(co, H * W).clone()
    p = torch.nn.functional.pad(x, (k // 2,) * 4)
    for dy in range(k):
        for dx in range(k):
            y.addmm_(w[:, :, dy, dx].contiguous(), p[:, dy:dy + H, dx:dx + W].reshape(C, H * W))
    return y.reshape(co, H, W)


def exact(case, seed):
    """The U-Net in float64.  Keys, depths and colours of a projection are copies of the cloud's values or
    selections by a float32 rule, and have no other value; served and whole frames start from them."""
    if case["kind"] != "unet":
        return None
    depth, rgba = _picture(case, seed)
    c, A = rgba.double(), rgba[..., 3].double()
    x = torch.stack([c[..., 0] / 255, c[..., 1] / 255, c[..., 2] / 255, A * depth.double() / 16, A])
    widths = _widths(case)
    ws = iter(_weights(widths, seed))
    skips = []
    for l in range(len(widths)):
        if l:
            x = torch.nn.functional.max_pool2d(x[None], 2)[0]
        for _ in (0, 1):
            x = _conv64(x, *next(ws)).clamp_(min=0)
        skips.append(x)
    for l in range(len(widths) - 2, -1, -1):
        x = torch.cat([skips[l], x.repeat_interleave(2, 1).repeat_interleave(2, 2)])
        for _ in (0, 1):
            x = _conv64(x, *next(ws)).clamp_(min=0)
    return _conv64(x, *next(ws))

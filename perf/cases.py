"""The measured work: tracking frames, image pyramids, ORB extraction and map edits as a user's program calls them.

Every case goes through `paper_2509_10757_amd.binding` (the C entry points with device tensors).  Inputs are synthetic
frames shaped like EuRoC (pinhole, 752x480) and TUM-VI (fisheye, 512x512) sequences, made from the seed alone: textured
stereo images, keypoints with the ORB per-level budget of which 80% are true pairs, descriptors with 0-24 flipped bits,
and local maps of points behind those keypoints plus uniform or clustered ones.  The sizes are those of the repository's
workloads (300-3000 keypoints per image, 1000-40000 map points, batches of up to 64 frames).
"""
from __future__ import annotations

import collections
import math

import numpy as np
import torch

from paper_2509_10757_amd import binding as ft

LEVELS = 8
BORDER = 16
MAX_KP, MAX_MAP, MAX_FRAMES, INFLIGHT = 4096, 65536, 64, 8


# ------------------------------------------------------------------ the cases
def listed():
    return [
        # one camera's frame, call by call: stereo, then the local-map search gated by its right coordinates
        {"name": "pinhole_300", "kind": "pinhole", "kp": 300, "map": 1000},       # few features: latency and launches
        {"name": "pinhole_1200", "kind": "pinhole", "kp": 1200, "map": 3000},     # the usual EuRoC frame
        {"name": "fisheye_1500", "kind": "fisheye", "kp": 1500, "map": 5000},     # the usual TUM-VI frame: both views
        # local-map search alone
        {"name": "clustered_20000", "kind": "search", "kp": 3000, "map": 20000, "fisheye": False, "clustered": True},
        {"name": "fisheye_map_39999", "kind": "search", "kp": 1533, "map": 39999, "fisheye": True, "clustered": False},
        # initial pose estimation: the last frame's matched points in the current frame
        {"name": "last_frame_1153", "kind": "last", "kp": 1200, "points": 1153, "direction": 0},
        # extraction: the pyramid of one image (a larger camera, odd sizes and pitch), corners and descriptors
        {"name": "pyramid_1281x719", "kind": "pyramid", "width": 1281, "height": 719, "pitch": 1283},
        {"name": "orb_752x480", "kind": "orb", "width": 752, "height": 480, "blur": 1.5},    # texture rich in corners
        {"name": "orb_511x509", "kind": "orb", "width": 511, "height": 509, "blur": 4.0},    # smoother: fewer corners
        # many cameras' frames in one submission; a small one whose pyramids are built on the device first
        {"name": "batch_64", "kind": "batch", "frames": 64, "kp_lo": 300, "kp_hi": 3000, "map_lo": 1000,
         "map_hi": 20000, "pinhole_share": 0.5, "images": False},
        {"name": "batch_8_images", "kind": "batch", "frames": 8, "kp_lo": 800, "kp_hi": 1600, "map_lo": 2000,
         "map_hi": 8000, "pinhole_share": 1.0, "images": True},
        # the local map edited in place: 5 % of it replaced, as between two frames
        {"name": "map_edit_20000", "kind": "edit", "map": 20000, "replaced": 1000},
    ]


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["pinhole", "fisheye", "search", "last", "pyramid", "orb", "batch", "edit"])
    if kind in ("pinhole", "fisheye"):
        return {"kind": kind, "kp": log_int(300, 3000), "map": log_int(1000, 20000)}
    if kind == "search":
        return {"kind": kind, "kp": log_int(300, 3000), "map": log_int(1000, 40000), "fisheye": rng.random() < 0.5,
                "clustered": rng.random() < 0.5}
    if kind == "last":
        kp = log_int(300, 3000)
        return {"kind": kind, "kp": kp, "points": int(rng.uniform(0.3, 1.0) * kp), "direction": rng.choice([-1, 0, 1])}
    if kind == "pyramid":
        w = log_int(320, 1536)
        return {"kind": kind, "width": w, "height": log_int(240, 1200), "pitch": w + rng.choice([0, 0, 1, 64])}
    if kind == "orb":
        return {"kind": kind, "width": log_int(320, 1000), "height": log_int(240, 600),
                "blur": rng.choice([1.5, 2.5, 4.0])}
    if kind == "batch":
        kp, mp = log_int(300, 1500), log_int(1000, 10000)
        return {"kind": kind, "frames": log_int(2, 48), "kp_lo": kp, "kp_hi": 2 * kp, "map_lo": mp, "map_hi": 2 * mp,
                "pinhole_share": rng.choice([0.0, 0.5, 1.0]), "images": rng.random() < 0.5}
    n = log_int(2000, 40000)
    return {"kind": kind, "map": n, "replaced": max(1, int(rng.uniform(0.01, 0.1) * n))}


# ------------------------------------------------------- what a program keeps
_ctx = None
_tickets = collections.deque()


def _context():
    """The program's one context, created at its start."""
    global _ctx
    if _ctx is None:
        _ctx = ft.Context(ft.default_limits(max_kp_per_image=MAX_KP, max_map_points=MAX_MAP, max_rows=1024,
                                            max_batch_frames=MAX_FRAMES, max_inflight=INFLIGHT,
                                            max_batch_kp_total=0, max_batch_map_total=0))
    return _ctx


# ------------------------------------------------------------------- scenes
def _scales():
    sf = np.empty(LEVELS, np.float32)
    sf[0] = 1.0
    for l in range(1, LEVELS):
        sf[l] = np.float32(sf[l - 1] * np.float32(1.2))
    return sf, (np.float32(1.0) / sf).astype(np.float32), (sf * sf).astype(np.float32)


SF, INV_SF, SIGMA2 = _scales()
WIDTH, HEIGHT, FX, CX, CY, BASE = 752, 480, 435.0, 367.0, 248.0, 0.11      # pinhole camera
BF = float(np.float32(np.float32(FX) * np.float32(BASE)))
FISH, FISH_F, FISH_BASE = 512, 190.0, 0.10                                   # fisheye cameras


def _scales_struct():
    s = ft.ft_scales()
    s.n_levels = LEVELS
    s.sf[:], s.inv_sf[:], s.sigma2[:] = [[float(v) for v in a] for a in (SF, INV_SF, SIGMA2)]
    return s


class Draws:
    """Seeded draws on the GPU, in 64 bits."""

    def __init__(self, seed):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(seed)

    def uni(self, lo, hi, *shape):
        return lo + (hi - lo) * torch.rand(*shape, generator=self.g, device="cuda", dtype=torch.float64)

    def normal(self, *shape):
        return torch.randn(*shape, generator=self.g, device="cuda", dtype=torch.float64)

    def ints(self, lo, hi, *shape):
        return torch.randint(lo, hi, shape, generator=self.g, device="cuda")

    def perm(self, n):
        return torch.argsort(torch.rand(n, generator=self.g, device="cuda", dtype=torch.float64))

    def bytes(self, n):
        return torch.randint(0, 256, (n, 32), generator=self.g, device="cuda", dtype=torch.uint8)

    def flipped(self, desc):
        """The same descriptors with about 0-24 flipped bits each."""
        n = desc.shape[0]
        p = self.uni(0.0, 24.0 / 256.0, n, 1)
        b = (self.uni(0.0, 1.0, n, 256) < p).view(n, 32, 8)
        w = torch.tensor([1, 2, 4, 8, 16, 32, 64, 128], device="cuda")
        return desc ^ (b * w).sum(2).to(torch.uint8)

    def levels(self, n):
        """Octaves with the ORB per-level budget, in random order."""
        share = np.cumsum([1.2 ** -l for l in range(LEVELS)])
        cut = torch.from_numpy(share / share[-1]).cuda()
        return torch.searchsorted(cut, self.uni(0.0, 1.0, n)).clamp_(max=LEVELS - 1)

    def unit(self, n):
        v = self.normal(n, 3)
        return v / v.norm(dim=1, keepdim=True)


def _sf64(l):
    return torch.from_numpy(SF.astype(np.float64)).cuda()[l]


def _texture(d, h, w, blur):
    r = int(math.ceil(4 * blur))
    k = torch.exp(-0.5 * (torch.arange(-r, r + 1, device="cuda", dtype=torch.float64) / blur) ** 2)
    k = k / k.sum()
    t = d.normal(h + 2 * r, w + 2 * r)
    t = sum(float(k[i]) * t[:, i:i + w] for i in range(2 * r + 1))
    t = sum(float(k[i]) * t[i:i + h] for i in range(2 * r + 1))
    t = (t - t.mean()) / t.std() * 45.0 + 128.0
    return t.round().clamp(0, 255)


class Disparity:
    """Eight planar facets of 2-60 px disparity."""

    def __init__(self, d):
        self.s = torch.stack([d.uni(0, WIDTH, 8), d.uni(0, HEIGHT, 8)])
        self.a, self.b, self.c = d.uni(2, 60, 8), d.uni(-0.03, 0.03, 8), d.uni(-0.03, 0.03, 8)

    def __call__(self, x, y):
        dx, dy = x[..., None] - self.s[0], y[..., None] - self.s[1]
        f = torch.argmin(dx * dx + dy * dy, dim=-1)
        return (self.a[f] + self.b[f] * (x - self.s[0][f]) + self.c[f] * (y - self.s[1][f])).clamp(2.0, 60.0)


def _pyramid(img, layout, total):
    """Every level bilinear from level 0, packed (the bytes a stereo call reads)."""
    out = torch.empty(total, dtype=torch.uint8, device="cuda")
    for l in range(LEVELS):
        w, h = layout.width[l], layout.height[l]
        lv = torch.nn.functional.interpolate(img[None, None], size=(h, w), mode="bilinear", align_corners=False)
        out[layout.offset[l]:layout.offset[l] + w * h] = lv.round().clamp(0, 255).to(torch.uint8).view(-1)
    return out


def _on_level(v, l):
    return (torch.round(v / _sf64(l)) * _sf64(l)).to(torch.float32)


def _map_fields(d, P, ref, desc):
    """Position, viewing normal within about 10 degrees, distance bounds that predict level `ref`, descriptor."""
    dist = P.norm(dim=1)
    nrm = P / dist[:, None] + 0.1 * d.unit(len(P)) * d.uni(0, 1, len(P), 1)
    nrm = nrm / nrm.norm(dim=1, keepdim=True)
    dmax = dist * _sf64(ref)
    o = d.perm(len(P))
    f = torch.float32
    return {"pos": P.to(f)[o].contiguous(), "normal": nrm.to(f)[o].contiguous(), "dmin": (dmax / float(SF[-1])).to(f)[o],
            "dmax": dmax.to(f)[o], "desc": desc[o].contiguous(), "order": o}


def _pose(d, R=np.eye(3), t=np.zeros(3)):
    """A pose 2 cm and 0.5 degrees off the frame's own (at the origin), moved into the camera (R, t)."""
    a = d.unit(2).cpu().numpy()
    k = np.array([[0, -a[0][2], a[0][1]], [a[0][2], 0, -a[0][0]], [-a[0][1], a[0][0], 0]])
    th = math.radians(0.5)
    R1 = np.eye(3) + math.sin(th) * k + (1 - math.cos(th)) * k @ k
    t1 = -R1 @ (0.02 * a[1])
    R2, t2 = R @ R1, R @ t1 + t
    return R2, t2, -R2.T @ t2


def _camera(model, f, cx, cy, k, bf, bounds, pose):
    return ft.search_camera_struct({"model": model, "fx": f, "fy": f, "cx": cx, "cy": cy, "k": k, "bf": bf, "R": pose[0],
                                    "t": pose[1], "O": pose[2], "bounds": bounds})


def _kps(x, y, octave, desc):
    return {"x": x.contiguous(), "y": y.contiguous(), "octave": octave.to(torch.uint8).contiguous(), "desc": desc.contiguous()}


def _pinhole_points(d, n):
    """n points of the pinhole view at 1-15 m: pixel, position."""
    u, v, z = d.uni(0, WIDTH, n), d.uni(0, HEIGHT, n), d.uni(1, 15, n)
    return torch.stack([(u - CX) * z / FX, (v - CY) * z / FX, z], 1)


def _pinhole(d, n_kp, n_map, images):
    """A rectified stereo frame: keypoints of both images, images (when wanted), the local map, the search camera."""
    field = Disparity(d)
    n_true = int(0.8 * n_kp)
    lv = d.levels(n_kp)
    sf = _sf64(lv)
    xl = _on_level(d.uni(70, WIDTH - 50, n_kp), lv)
    yl = _on_level(d.uni(50, HEIGHT - 50, n_kp), lv)
    x, y = xl.double(), yl.double()
    xr = x - field(x, y)
    for _ in range(6):
        xr = x - field(xr, y)
    lr = torch.where(d.uni(0, 1, n_kp) < 0.85, lv, (lv + 2 * d.ints(0, 2, n_kp) - 1).clamp(0, LEVELS - 1))
    xr2, yr2 = _on_level(xr, lr), _on_level(y + d.ints(-1, 2, n_kp) * _sf64(lr), lr)
    true = torch.arange(n_kp, device="cuda") < n_true
    xr2 = torch.where(true, xr2, _on_level(d.uni(20, WIDTH - 20, n_kp), lr))
    yr2 = torch.where(true, yr2, _on_level(d.uni(20, HEIGHT - 20, n_kp), lr))
    dl = d.bytes(n_kp)
    dr = torch.where(true[:, None], d.flipped(dl), d.bytes(n_kp))
    z = (BF / (x - xr).clamp(min=1.0)).clamp(1.0, 15.0)
    P = torch.stack([(x - CX) * z / FX, (y - CY) * z / FX, z], 1)
    n_from = min(n_true, n_map)
    pts = torch.cat([P[:n_from], _pinhole_points(d, n_map - n_from)])
    ref = torch.cat([lv[:n_from], d.ints(0, LEVELS, n_map - n_from)])
    mp = _map_fields(d, pts, ref, torch.cat([d.flipped(dl[:n_from]), d.bytes(n_map - n_from)]))
    pl, pr = d.perm(n_kp), d.perm(n_kp)
    f = {"kind": "pinhole", "left": _kps(xl[pl], yl[pl], lv[pl], dl[pl]), "right": _kps(xr2[pr], yr2[pr], lr[pr], dr[pr]),
         "map": mp, "views": [{"cam": _camera(0, FX, CX, CY, [0] * 4, BF, [0, WIDTH, 0, HEIGHT], _pose(d)), "grid": (64, 48),
                               "pre": (d.uni(0, 1, n_kp) < 0.1).to(torch.uint8)}],
         "true": (pl, n_from, (x - xr)[pl])}
    if images:
        left = _texture(d, HEIGHT, WIDTH, 1.5)
        ys, xs = torch.meshgrid(torch.arange(HEIGHT, device="cuda", dtype=torch.float64),
                                torch.arange(WIDTH, device="cuda", dtype=torch.float64), indexing="ij")
        src = xs + field(xs, ys)
        i = src.floor().clamp(max=WIDTH - 2).long()
        fr = src - i
        row = torch.arange(HEIGHT, device="cuda")[:, None]
        right = torch.where(src < WIDTH - 1, left[row, i] * (1 - fr) + left[row, i + 1] * fr, _texture(d, HEIGHT, WIDTH, 1.5))
        right = (right + 2.0 * d.normal(HEIGHT, WIDTH)).round().clamp(0, 255)
        f["images"] = (left, right)
    return f


def _kb_project(X, k):
    rho = torch.sqrt(X[:, 0] ** 2 + X[:, 1] ** 2)
    th = torch.atan2(rho, X[:, 2])
    t2 = th * th
    thd = th * ((((1.0 + float(k[0]) * t2) + float(k[1]) * t2 ** 2) + float(k[2]) * t2 ** 3) + float(k[3]) * t2 ** 4)
    s = torch.where(rho > 0, thd / rho, torch.zeros_like(rho))
    return FISH_F * X[:, 0] * s + FISH / 2, FISH_F * X[:, 1] * s + FISH / 2


def _cap(d, n, max_deg=75.0):
    """n points at 1-15 m with a ray angle of at most max_deg."""
    c, phi = d.uni(math.cos(math.radians(max_deg)), 1, n), d.uni(0, 2 * math.pi, n)
    s = torch.sqrt(1 - c * c)
    return torch.stack([s * torch.cos(phi), s * torch.sin(phi), c], 1) * d.uni(1, 15, n, 1)


def _fisheye(d, n_kp, n_map):
    kl, kr = [np.float32(d.uni(-0.01, 0.01, 4).cpu().numpy()) for _ in range(2)]
    a = math.radians(2.0)
    R_lr = np.array([[math.cos(a), 0, math.sin(a)], [0, 1, 0], [-math.sin(a), 0, math.cos(a)]])
    t_lr = np.array([FISH_BASE, 0, 0])
    R_rl, t_rl = R_lr.T, -R_lr.T @ t_lr
    n_true = int(0.8 * n_kp)
    X = _cap(d, n_kp, 70.0)
    Xr = X @ torch.from_numpy(R_rl.T).cuda() + torch.from_numpy(t_rl).cuda()
    lv = d.levels(n_kp)
    lr = torch.where(d.uni(0, 1, n_kp) < 0.85, lv, (lv + 2 * d.ints(0, 2, n_kp) - 1).clamp(0, LEVELS - 1))
    true = torch.arange(n_kp, device="cuda") < n_true
    xy = []
    for P, l, k in ((X, lv, kl), (Xr, lr, kr)):
        u, v = _kb_project(P, k)
        u = torch.where(true, u, d.uni(BORDER, FISH - BORDER, n_kp))
        v = torch.where(true, v, d.uni(BORDER, FISH - BORDER, n_kp))
        xy.append([_on_level(c.clamp(BORDER, FISH - BORDER), l) for c in (u, v)])
    dl = d.bytes(n_kp)
    dr = torch.where(true[:, None], d.flipped(dl), d.bytes(n_kp))
    n_from = min(n_true, n_map)
    pts = torch.cat([X[:n_from], _cap(d, n_map - n_from)])
    ref = torch.cat([lv[:n_from], d.ints(0, LEVELS, n_map - n_from)])
    mp = _map_fields(d, pts, ref, torch.cat([d.flipped(dl[:n_from]), d.bytes(n_map - n_from)]))
    pl, pr = d.perm(n_kp), d.perm(n_kp)
    cam = ft.ft_fisheye_stereo()
    for side, k in ((cam.left, kl), (cam.right, kr)):
        side.fx, side.fy, side.cx, side.cy = FISH_F, FISH_F, FISH / 2, FISH / 2
        side.k[:] = [float(v) for v in k]
    cam.R_lr[:] = [float(np.float32(v)) for v in R_lr.reshape(-1)]
    cam.t_lr[:] = [float(np.float32(v)) for v in t_lr]
    cam.overlap_left[:] = [float(np.float32(0.4 * FISH)), float(FISH)]
    cam.overlap_right[:] = [0.0, float(np.float32(0.6 * FISH))]
    R, t, _ = p = _pose(d)
    q = (R_rl @ R, R_rl @ t + t_rl)
    views = [{"cam": _camera(1, FISH_F, FISH / 2, FISH / 2, k, 0.0, [0, FISH, 0, FISH], pose), "grid": (64, 48),
              "pre": (d.uni(0, 1, n_kp) < 0.1).to(torch.uint8)}
             for k, pose in ((kl, p), (kr, (q[0], q[1], -q[0].T @ q[1])))]
    return {"kind": "fisheye", "left": _kps(xy[0][0][pl], xy[0][1][pl], lv[pl], dl[pl]),
            "right": _kps(xy[1][0][pr], xy[1][1][pr], lr[pr], dr[pr]), "map": mp, "views": views, "stereo_cam": cam}


def _clustered(d, n_kp, n_map, fisheye):
    """A map in 40 blobs (sigma 0.5 m) and a frame of which 80% of the keypoints are its projections."""
    centres = _cap(d, 40, 60.0) if fisheye else _pinhole_points(d, 40)
    P = centres[d.ints(0, 40, n_map)] + 0.5 * d.normal(n_map, 3)
    P[:, 2] = P[:, 2].clamp(min=0.8)
    kb = np.float32(d.uni(-0.01, 0.01, 4).cpu().numpy()) if fisheye else np.zeros(4, np.float32)
    W, H = (FISH, FISH) if fisheye else (WIDTH, HEIGHT)
    ref = d.ints(0, LEVELS, n_map)
    desc = d.bytes(n_map)
    src = d.ints(0, n_map, n_kp)
    lv = (ref[src] + d.ints(-1, 2, n_kp)).clamp(0, LEVELS - 1)
    if fisheye:
        u, v = _kb_project(P[src], kb)
    else:
        u, v = FX * P[src][:, 0] / P[src][:, 2] + CX, FX * P[src][:, 1] / P[src][:, 2] + CY
    other = d.uni(0, 1, n_kp) < 0.2
    u, v = torch.where(other, d.uni(0, W, n_kp), u), torch.where(other, d.uni(0, H, n_kp), v)
    kd = torch.where(other[:, None], d.bytes(n_kp), d.flipped(desc[src]))
    kps = _kps(_on_level(u, lv).clamp(0, W - 1), _on_level(v, lv).clamp(0, H - 1), lv, kd)
    cam = _camera(1, FISH_F, W / 2, H / 2, kb, 0.0, [0, W, 0, H], _pose(d)) if fisheye else \
        _camera(0, FX, CX, CY, kb, BF, [0, W, 0, H], _pose(d))
    return {"kind": "search", "left": kps, "map": _map_fields(d, P, ref, desc),
            "views": [{"cam": cam, "grid": (96, 64), "pre": torch.zeros(n_kp, dtype=torch.uint8, device="cuda")}]}


# ------------------------------------------------- device arrays and structs
def _kp_struct(k):
    return ft.ft_keypoints(len(k["x"]), k["x"].data_ptr(), k["y"].data_ptr(), k["octave"].data_ptr(), k["desc"].data_ptr())


def _map_struct(m):
    return ft.ft_map_points(len(m["dmin"]), m["pos"].data_ptr(), m["normal"].data_ptr(), m["dmin"].data_ptr(),
                            m["dmax"].data_ptr(), m["desc"].data_ptr())


PINHOLE_PARAMS = (75, 5, 5, 1, 21, 10, 2.0)
SEARCH_PARAMS = (2.0, 0.5, 0.998, 2.5, 4.0, 0.8, 1.2, 1, 1, 100, 4, 5, 1)


def _layout():
    return ft.pyramid_layout(WIDTH, HEIGHT, _scales_struct())


class Frames:
    """Frames with their outputs in shared arenas (each output array of all frames end to end) and their structs."""

    def __init__(self, frames, build_images=False):
        self.frames, self.build = frames, build_images
        self.scales = _scales_struct()
        self.search_params = ft.ft_search_params(*SEARCH_PARAMS)
        i32, f32 = torch.int32, torch.float32
        n_l = sum(len(f["left"]["x"]) for f in frames)
        n_v = sum(len(f["views"]) for f in frames)
        n_m = sum(len(f["views"]) * len(f["map"]["dmin"]) for f in frames)
        n_k = sum(len(f["left" if v == 0 else "right"]["x"]) for f in frames for v in range(len(f["views"])))
        new = lambda dt, *s: torch.zeros(s, dtype=dt, device="cuda")  # noqa: E731
        self.out = {"mp_match": new(i32, n_m), "mp_dist": new(i32, n_m), "kp_match": new(i32, n_k),
                    "search_n": new(i32, n_v)}
        kinds = {f["kind"] for f in frames}
        if kinds & {"pinhole", "fisheye"}:
            self.out |= {"right_idx": new(i32, n_l), "dist": new(i32, n_l), "depth": new(f32, n_l),
                         "stereo_n": new(i32, len(frames))}
        if "pinhole" in kinds:
            self.out |= {"u_right": new(f32, n_l), "sad": new(i32, n_l)}
            lay, total = _layout()
            n_pyr = 2 * sum(f["kind"] == "pinhole" for f in frames)
            self.pyr = torch.zeros((n_pyr, total), dtype=torch.uint8, device="cuda")
            if build_images:
                self.out["pyramids"] = self.pyr
        if "fisheye" in kinds:
            self.out["xyz"] = new(f32, n_l, 3)
        self.items = []
        at = dict(l=0, v=0, m=0, k=0, p=0)
        for i, f in enumerate(frames):
            self.items.append(self._item(i, f, at))
        if len(frames) > 1 or build_images:
            self.jobs = (ft.ft_frame_job * len(frames))(*[self._job(i) for i in range(len(frames))])

    def _p(self, name, i):
        t = self.out[name]
        return t.data_ptr() + i * t.element_size() * (3 if name == "xyz" else 1)

    def _item(self, i, f, at):
        it = {"left": _kp_struct(f["left"]), "map": _map_struct(f["map"]), "views": []}
        l = at["l"]
        if f["kind"] != "search":
            it["right"] = _kp_struct(f["right"])
        if f["kind"] == "pinhole":
            pyr = []
            f["img_u8"] = [im.to(torch.uint8).contiguous() for im in f["images"]]
            for im in f["images"]:
                s, total = _layout()
                s.data = self.pyr[at["p"]].data_ptr()
                if not self.build:
                    self.pyr[at["p"]] = _pyramid(im, s, total)
                pyr.append(s)
                at["p"] += 1
            it["pyr"] = pyr
            it["cam"] = ft.ft_pinhole_stereo(FX, BF, BASE, HEIGHT)
            it["params"] = ft.ft_pinhole_params(*PINHOLE_PARAMS)
            it["out"] = ft.ft_pinhole_out(*[self._p(n, l) for n in ("right_idx", "dist", "u_right", "depth", "sad")],
                                          self._p("stereo_n", i))
        elif f["kind"] == "fisheye":
            it["cam"] = f["stereo_cam"]
            it["params"] = ft.ft_fisheye_params(7, 10, 10, 0, 0.9998, 5.991, math.radians(88.0), 1e-12)
            it["out"] = ft.ft_fisheye_out(*[self._p(n, l) for n in ("right_idx", "dist", "depth", "xyz")], self._p("stereo_n", i))
        for v, spec in enumerate(f["views"]):
            it["views"].append(ft.ft_search_out(self._p("mp_match", at["m"]), self._p("mp_dist", at["m"]),
                                                self._p("kp_match", at["k"]), self._p("search_n", at["v"])))
            at["m"] += len(f["map"]["dmin"])
            at["k"] += len(f["left" if v == 0 else "right"]["x"])
            at["v"] += 1
        at["l"] += len(f["left"]["x"])
        return it

    def _job(self, i):
        f, it, j = self.frames[i], self.items[i], ft.ft_frame_job()
        j.kind = ft.FT_JOB_PINHOLE if f["kind"] == "pinhole" else ft.FT_JOB_FISHEYE
        j.n_views = len(f["views"])
        j.left, j.right, j.scales, j.map = it["left"], it["right"], self.scales, it["map"]
        j.search_params = self.search_params
        if f["kind"] == "pinhole":
            j.pyr_left, j.pyr_right = it["pyr"]
            j.pinhole, j.pinhole_params, j.pinhole_out, j.use_u_right = it["cam"], it["params"], it["out"], 1
            if self.build:
                j.build_pyramids = 1
                j.image_left, j.image_right = [ft.ft_image(t.data_ptr(), WIDTH, HEIGHT, WIDTH) for t in f["img_u8"]]
        else:
            j.fisheye, j.fisheye_params, j.fisheye_out = it["cam"], it["params"], it["out"]
        for v, spec in enumerate(f["views"]):
            j.cam[v], j.grid[v], j.search_out[v] = spec["cam"], ft.ft_grid(*spec["grid"]), it["views"][v]
            j.preassigned[v] = spec["pre"].data_ptr()
        return j

    def calls(self):
        """The single frame's calls with their arguments."""
        f, it = self.frames[0], self.items[0]
        todo, u_right = [], None
        if f["kind"] == "pinhole":
            todo.append(("ft_stereo_match_pinhole", (it["left"], it["right"], it["pyr"][0], it["pyr"][1], self.scales, it["cam"],
                                                     it["params"], it["out"])))
            u_right = self._p("u_right", 0)
        elif f["kind"] == "fisheye":
            todo.append(("ft_stereo_match_fisheye", (it["left"], it["right"], self.scales, it["cam"], it["params"], it["out"])))
        for v, spec in enumerate(f["views"]):
            todo.append(("ft_search_local_points", (it["map"], spec["cam"], it["left" if v == 0 else "right"], u_right,
                                                    spec["pre"].data_ptr(), ft.ft_grid(*spec["grid"]), self.scales,
                                                    self.search_params, it["views"][v])))
        return todo


def _frames(case, seed):
    d = Draws(seed)
    kind = case["kind"]
    if kind == "pinhole":
        return [_pinhole(d, case["kp"], case["map"], True)]
    if kind == "fisheye":
        return [_fisheye(d, case["kp"], case["map"])]
    if kind == "search":
        if case["clustered"]:
            return [_clustered(d, case["kp"], case["map"], case["fisheye"])]
        f = _fisheye(d, case["kp"], case["map"]) if case["fisheye"] else _pinhole(d, case["kp"], case["map"], False)
        return [{"kind": "search", "left": f["left"], "map": f["map"], "views": f["views"][:1]}]
    # the frames' sizes are the case's, their contents the seed's
    n, r = case["frames"], np.random.RandomState(case["frames"] + case["kp_lo"])
    pin = r.permutation(n) < round(case["pinhole_share"] * n)
    kp = [int(v) for v in r.randint(case["kp_lo"], case["kp_hi"] + 1, n)]
    mp = [int(v) for v in r.randint(case["map_lo"], case["map_hi"] + 1, n)]
    return [_pinhole(d, kp[i], mp[i], True) if pin[i] else _fisheye(d, kp[i], mp[i]) for i in range(n)]


def _last(case, seed):
    """The last frame's matched points: 80% behind current keypoints, their octave moved by one now and then."""
    d = Draws(seed)
    f = _pinhole(d, case["kp"], max(case["kp"], case["points"]), False)
    n, mp, kp = case["points"], f["map"], f["left"]
    pl, n_from, disp = f["true"]
    inv = torch.empty_like(pl)
    inv[pl] = torch.arange(len(pl), device="cuda")
    owner = mp["order"]                                   # map point -> generated point
    is_true = owner < n_from
    k_of = inv[owner.clamp(max=len(pl) - 1)]
    pick = torch.argsort(d.uni(0, 1, len(owner)) + 10.0 * (~is_true))[:n]
    pick = pick[d.perm(n)]
    t, k = is_true[pick], k_of[pick]
    octave = torch.where(t, kp["octave"].long()[k], d.ints(0, LEVELS, n))
    octave = (octave + torch.where(d.uni(0, 1, n) < 0.3, 2 * d.ints(0, 2, n) - 1, 0)).clamp(0, LEVELS - 1)
    angle = d.uni(0, 360, n)
    ka = d.uni(0, 360, len(kp["x"]))
    tt = t & (d.uni(0, 1, n) < 0.9)
    ka[k[tt]] = (angle - 5.0 + 3.0 * d.normal(n))[tt] % 360.0
    u_r = torch.full((len(kp["x"]),), -1.0, dtype=torch.float32, device="cuda")
    kt = k[t]
    u_r[kt] = (kp["x"].double()[kt] - disp[kt] + d.uni(-0.3, 0.3, len(kt))).float()
    return {"pos": mp["pos"][pick].contiguous(), "desc": mp["desc"][pick].contiguous(), "octave": octave.to(torch.uint8),
            "angle": angle.float(), "kps": kp, "kp_angle": ka.float(), "u_right": u_r, "view": f["views"][0]}


def _pattern():
    """256 pairs of points within radius 13, isotropic Gaussian with sigma 31/5."""
    r = np.random.RandomState(31)
    p = np.rint(r.normal(0.0, 31 / 5.0, (20000, 2)))
    p = p[(p ** 2).sum(1) <= 169].astype(np.int8)
    return np.ascontiguousarray(p[:2 * 256].reshape(256, 4))


def _edit_inputs(case, seed):
    d = Draws(seed)
    n, m = case["map"], case["replaced"]
    maps = []
    for k in (n, m):
        P = _pinhole_points(d, k)
        maps.append(_map_fields(d, P, d.ints(0, LEVELS, k), d.bytes(k)))
    return maps[0], maps[1], d.perm(n)[:m].cpu().numpy().astype(np.int32)


# -------------------------------------------------------------- prepare, run
def prepare(case, seed):
    kind, ctx = case["kind"], _context()
    if kind in ("pinhole", "fisheye", "search"):
        fr = Frames(_frames(case, seed))
        return {"kind": "calls", "calls": [(getattr(ctx, name), args) for name, args in fr.calls()], "out": fr.out, "keep": fr}
    if kind == "batch":
        fr = Frames(_frames(case, seed), case["images"] and case["pinhole_share"] > 0)
        if not hasattr(fr, "jobs"):
            raise ValueError("a batch has at least two frames")
        return {"kind": "batch", "addr": ft.ct.addressof(fr.jobs), "n": case["frames"], "out": fr.out, "keep": fr}
    if kind == "last":
        c = _last(case, seed)
        n, k = case["points"], c["kps"]
        z = lambda n: torch.zeros(n, dtype=torch.int32, device="cuda")  # noqa: E731
        out = {"mp_match": z(n), "mp_dist": z(n), "kp_match": z(len(k["x"])), "n_matches": z(1)}
        last = ft.ft_last_points(n, c["pos"].data_ptr(), c["desc"].data_ptr(), c["octave"].data_ptr(), c["angle"].data_ptr())
        args = (last, c["view"]["cam"], _kp_struct(k), c["kp_angle"].data_ptr(), c["u_right"].data_ptr(),
                c["view"]["pre"].data_ptr(), ft.ft_grid(*c["view"]["grid"]), _scales_struct(),
                ft.ft_last_params(7.0, 100, case["direction"], 1, 30), ft.ft_search_out(*[t.data_ptr() for t in out.values()]))
        return {"kind": "calls", "calls": [(ctx.ft_search_last_frame, args)], "out": out, "keep": c}
    if kind == "pyramid":
        w, h, pitch = case["width"], case["height"], case["pitch"]
        img = torch.zeros((h, pitch), dtype=torch.uint8, device="cuda")
        img[:, :w] = _texture(Draws(seed), h, w, 1.5).to(torch.uint8)
        lay, total = ft.pyramid_layout(w, h, _scales_struct())
        out = torch.zeros(total, dtype=torch.uint8, device="cuda")
        lay.data = out.data_ptr()
        args = (ft.ft_image(img.data_ptr(), w, h, pitch), _scales_struct(), lay)
        return {"kind": "calls", "calls": [(ctx.ft_build_pyramid, args)], "out": {"pyramid": out}, "keep": img}
    if kind == "orb":
        data, lay = _orb_pyramid(case, seed)
        lay.data = data.data_ptr()
        c = 65536
        z = lambda dt, *s: torch.zeros(s, dtype=dt, device="cuda")  # noqa: E731
        out = {"lx": z(torch.int16, c), "ly": z(torch.int16, c), "octave": z(torch.uint8, c), "score": z(torch.uint8, c),
               "x": z(torch.float32, c), "y": z(torch.float32, c), "count": z(torch.int32, 1), "angle": z(torch.float32, c),
               "desc": z(torch.uint8, c, 32), "blurred": torch.zeros_like(data)}
        p = {k: t.data_ptr() for k, t in out.items()}
        corners = ft.ft_orb_corners(c, p["lx"], p["ly"], p["octave"], p["score"], p["x"], p["y"], p["count"])
        sc = _scales_struct()
        return {"kind": "calls", "out": out, "keep": data, "calls": [
            (ctx.ft_orb_detect, (lay, sc, ft.ft_orb_params(20, 19), p["blurred"], corners)),
            (ctx.ft_orb_describe, (lay, p["blurred"], c, p["count"], p["lx"], p["ly"], p["octave"], _pattern(), p["angle"],
                                   p["desc"]))]}
    mp, ins, rem = _edit_inputs(case, seed)
    out = {k: v for k, v in mp.items() if k != "order"}
    return {"kind": "calls", "calls": [(ctx.ft_map_update, (_map_struct(mp), case["map"], rem, _map_struct(ins)))], "out": out,
            "keep": (mp, ins)}


def run(state):
    if state["kind"] == "batch":
        while len(_tickets) >= INFLIGHT:
            _ctx.ft_batch_wait(_tickets.popleft())
        _tickets.append(_ctx.ft_batch_submit_raw(state["addr"], state["n"]))
    else:
        for fn, args in state["calls"]:
            fn(*args)
    return state["out"]


# ---------------------------------------------------------------------- work
def _pyramid_bytes(w, h):
    lay, total = ft.pyramid_layout(w, h, _scales_struct())
    return total


def _frame_work(kind, kp, mp, images=False):
    b = f = 0
    views = {"pinhole": 1, "search": 1, "fisheye": 2}[kind]
    if kind == "pinhole":                                  # both images' keypoints, 80% refined windows, outputs
        b += 82 * kp + 0.8 * kp * (121 + 231) + 20 * kp
        f += 0.8 * kp * 11 * 121 * 3
        if images:
            b += 2 * (WIDTH * HEIGHT + _pyramid_bytes(WIDTH, HEIGHT))
    elif kind == "fisheye":                                # all pairs of the overlap (60% of the width): 256 terms each
        b += 82 * kp + 24 * kp
        f += 2 * 256 * (0.6 * kp) ** 2
    return b + views * (72 * mp + 50 * kp), f


def work(case):
    kind = case["kind"]
    if kind in ("pinhole", "fisheye", "search"):
        b, f = _frame_work(kind, case["kp"], case["map"])
    elif kind == "batch":
        kp, mp = (case["kp_lo"] + case["kp_hi"]) / 2, (case["map_lo"] + case["map_hi"]) / 2
        p, q = _frame_work("pinhole", kp, mp, case["images"]), _frame_work("fisheye", kp, mp)
        s = case["pinhole_share"]
        b, f = [case["frames"] * (s * x + (1 - s) * y) for x, y in zip(p, q)]
    elif kind == "last":
        b, f = (12 + 32 + 5 + 8) * case["points"] + 58 * case["kp"], 0
    elif kind == "pyramid":
        b, f = case["width"] * case["height"] + _pyramid_bytes(case["width"], case["height"]), 0
    elif kind == "orb":                                    # pyramid read, smoothed one written; per corner 50 bytes
        n = _pyramid_bytes(case["width"], case["height"])
        b, f = 2 * n + 50 * n * {1.5: 0.043, 2.5: 0.018, 4.0: 0.007}[case["blur"]], 0
    else:
        b, f = 2 * 64 * 2 * case["replaced"], 0
    return {"bytes": float(b), "flops": float(f)}


# ------------------------------------------------- the same in 64 bits, plain
def _orb_pyramid(case, seed):
    lay, total = ft.pyramid_layout(case["width"], case["height"], _scales_struct())
    return _pyramid(_texture(Draws(seed), case["height"], case["width"], case["blur"]), lay, total), lay


def _built_pyramid(img, layout, total):
    """Every level from level 0 as ft_build_pyramid defines it: source coordinates as exact fractions, 8-bit weights."""
    out = torch.empty(total, dtype=torch.uint8, device="cuda")
    img = img.long()

    def taps(n_in, n):
        num = (2 * torch.arange(n, device="cuda") + 1) * n_in - n
        q, w = num // (2 * n), num % (2 * n) * 256 // (2 * n)
        w = torch.where((q < 0) | (q >= n_in - 1), 0, w)
        q = q.clamp(0, n_in - 1)
        return q, (q + 1).clamp(max=n_in - 1), w

    for l in range(LEVELS):
        w, h = layout.width[l], layout.height[l]
        y0, y1, b = taps(img.shape[0], h)
        x0, x1, a = taps(img.shape[1], w)
        rows = img[y0] * (256 - b)[:, None] + img[y1] * b[:, None]
        v = rows[:, x0] * (256 - a) + rows[:, x1] * a
        out[layout.offset[l]:layout.offset[l] + w * h] = ((v + 32768) >> 16).to(torch.uint8).view(-1)
    return out


def _hamming(a, b):
    def signs(t):
        w = torch.tensor([1, 2, 4, 8, 16, 32, 64, 128], device="cuda", dtype=torch.uint8)
        return ((t[:, :, None] & w) != 0).view(len(t), 256).double() * 2 - 1
    return ((256 - signs(a) @ signs(b).T) / 2).round().long()


def _winners(take, h, i, j, n_right):
    """Of the taken matches of one right keypoint, the smallest (distance, left index)."""
    key = torch.where(take, h * (1 << 23) + i, torch.full_like(h, 1 << 60))
    best = torch.full((n_right,), 1 << 60, device="cuda", dtype=torch.int64).scatter_reduce(0, j, key, "amin")
    return take & (best[j] == key)


def _exact_pinhole(f, pyr):
    """(u_right, depth) of a pinhole frame: row band and levels decided on the given binary32 values, the rest in 64 bits."""
    L, R = f["left"], f["right"]
    n = len(L["x"])
    sf = torch.from_numpy(SF).cuda()
    ol, orr = L["octave"].long(), R["octave"].long()
    r = 2.0 * sf[orr]
    lo, hi = (R["y"] - r).floor().clamp(min=0), (R["y"] + r).ceil().clamp(max=HEIGHT - 1)
    row = L["y"].trunc()
    maxd = float(np.float32(np.float32(BF) / np.float32(BASE)))
    cand = (row[:, None] >= lo) & (row[:, None] <= hi) & ((ol[:, None] - orr).abs() <= 1) & \
        (R["x"] >= (L["x"] - maxd)[:, None]) & (R["x"] <= L["x"][:, None]) & (L["y"] < HEIGHT)[:, None]
    key = torch.where(cand, _hamming(L["desc"], R["desc"]) * 65536 + torch.arange(len(R["x"]), device="cuda"), 1 << 40)
    best = key.min(1).values
    h, j = best >> 16, torch.where(best < (1 << 40), best & 65535, 0)
    ok = h < 75
    s = torch.from_numpy(INV_SF).cuda().double()[ol]
    up = lambda v: torch.floor(v * s + 0.5).long()  # noqa: E731
    su, sv, sr = up(L["x"].double()), up(L["y"].double()), up(R["x"].double()[j])
    lay, _ = _layout()
    w, hh, off = [torch.tensor(list(v), device="cuda")[ol] for v in (lay.width, lay.height, lay.offset)]
    ok &= (su >= 5) & (su + 5 < w) & (sv >= 5) & (sv + 5 < hh) & (sr >= 10) & (sr + 10 < w)
    d = torch.arange(-5, 6, device="cuda")
    at = lambda x, y: off[:, None, None] + y * w[:, None, None] + x  # noqa: E731
    yy = (sv[:, None, None] + d[None, :, None])
    zero = torch.zeros((), dtype=torch.int64, device="cuda")
    keep = ok[:, None, None]
    a = pyr[0].long()[torch.where(keep, at(su[:, None, None] + d, yy), zero)]
    b = pyr[1].long()[torch.where(keep, at(sr[:, None, None] + torch.arange(-10, 11, device="cuda"), yy), zero)]
    a = a - a[:, 5:6, 5:6]
    sad = torch.stack([(a - (b[:, :, k:k + 11] - b[:, 5:6, k + 5:k + 6])).abs().sum((1, 2)) for k in range(11)], 1)
    c, k = sad.min(1)
    k = (sad == c[:, None]).long().argmax(1)
    ok &= (k > 0) & (k < 10)
    m = sad.gather(1, torch.stack([(k - 1).clamp(min=0), (k + 1).clamp(max=10)], 1)).double()
    delta = (m[:, 0] - m[:, 1]) / (2 * (m[:, 0] + m[:, 1] - 2 * c.double()))
    ok &= delta.abs() <= 1
    x = L["x"].double()
    ur = sf.double()[ol] * (sr + k - 5 + delta)
    disp = x - ur
    ok &= (disp >= 0) & (disp < maxd)
    ur, disp = torch.where(disp <= 0, x - 0.01, ur), torch.where(disp <= 0, 0.01, disp)
    ok = _winners(ok, h, torch.arange(n, device="cuda"), j, len(R["x"]))
    if int(ok.sum()):
        med = c[ok].sort().values[int(ok.sum()) // 2]
        ok &= 10 * c < 21 * med
    return torch.where(ok, ur, -1.0), torch.where(ok, BF / disp, -1.0)


def _exact_fisheye(f):
    """(depth, xyz) of a fisheye frame in 64 bits."""
    L, R, cam = f["left"], f["right"], f["stereo_cam"]
    n = len(L["x"])
    q = ((L["x"] >= cam.overlap_left[0]) & (L["x"] <= cam.overlap_left[1])).nonzero().view(-1)
    t = ((R["x"] >= cam.overlap_right[0]) & (R["x"] <= cam.overlap_right[1])).nonzero().view(-1)
    depth = torch.full((n,), -1.0, dtype=torch.float64, device="cuda")
    xyz = torch.zeros((n, 3), dtype=torch.float64, device="cuda")
    if len(t) < 2 or not len(q):
        return depth, xyz
    two = (_hamming(L["desc"][q], R["desc"][t]) * 65536 + t).sort(1).values[:, :2]
    h, j = two[:, 0] >> 16, two[:, 0] & 65535
    ok = 10 * h < 7 * (two[:, 1] >> 16)

    def ray(c, x, y):
        k = [float(v) for v in c.k]
        xp, yp = (x.double() - c.cx) / c.fx, (y.double() - c.cy) / c.fy
        thd = torch.sqrt(xp * xp + yp * yp).clamp(max=math.pi / 2)
        th = thd.clone()
        live = torch.ones_like(th, dtype=torch.bool)
        for _ in range(10):
            t2 = th * th
            g = th * (1 + k[0] * t2 + k[1] * t2 ** 2 + k[2] * t2 ** 3 + k[3] * t2 ** 4) - thd
            gp = 1 + 3 * k[0] * t2 + 5 * k[1] * t2 ** 2 + 7 * k[2] * t2 ** 3 + 9 * k[3] * t2 ** 4
            step = torch.where(live, g / gp, torch.zeros_like(g))
            th = th - step
            live &= step.abs() >= 1e-12
        small = thd <= 1e-8
        sc = torch.where(small, torch.ones_like(th), torch.tan(th) / torch.where(small, torch.ones_like(thd), thd))
        return torch.stack([xp * sc, yp * sc, torch.ones_like(xp)], 1), small | (th < math.radians(88.0))

    Rm = torch.tensor(list(cam.R_lr), dtype=torch.float64, device="cuda").view(3, 3)
    tv = torch.tensor(list(cam.t_lr), dtype=torch.float64, device="cuda")
    r1, ok1 = ray(cam.left, L["x"][q], L["y"][q])
    r2, ok2 = ray(cam.right, R["x"][j], R["y"][j])
    ok &= ok1 & ok2
    r21 = r2 @ Rm.T
    ok &= (r1 * r21).sum(1) / (r1.norm(dim=1) * r21.norm(dim=1)) <= 0.9998
    Rr, tr = Rm.T, -(Rm.T @ tv)
    A = torch.zeros((len(q), 4, 3), dtype=torch.float64, device="cuda")
    A[:, 0, 0] = A[:, 1, 1] = -1.0
    A[:, 0, 2], A[:, 1, 2] = r1[:, 0], r1[:, 1]
    A[:, 2] = r2[:, :1] * Rr[2] - Rr[0]
    A[:, 3] = r2[:, 1:2] * Rr[2] - Rr[1]
    b = torch.zeros((len(q), 4), dtype=torch.float64, device="cuda")
    b[:, 2], b[:, 3] = -(r2[:, 0] * tr[2] - tr[0]), -(r2[:, 1] * tr[2] - tr[1])
    M = (A[:, :, :, None] * A[:, :, None, :]).sum(1)
    v = (A * b[:, :, None]).sum(1)

    def det(m):
        return m[:, 0, 0] * (m[:, 1, 1] * m[:, 2, 2] - m[:, 1, 2] * m[:, 2, 1]) - \
            m[:, 0, 1] * (m[:, 1, 0] * m[:, 2, 2] - m[:, 1, 2] * m[:, 2, 0]) + \
            m[:, 0, 2] * (m[:, 1, 0] * m[:, 2, 1] - m[:, 1, 1] * m[:, 2, 0])

    D = det(M)
    X = []
    for c in range(3):
        Mc = M.clone()
        Mc[:, :, c] = v
        X.append(det(Mc) / D)
    X = torch.stack(X, 1)
    X2 = (X - tv) @ Rm
    ok &= (X[:, 2] > 0) & (X2[:, 2] > 0)
    for P, c, K, idx in ((X, cam.left, L, q), (X2, cam.right, R, j)):
        u, w = _kb_project(P, list(c.k))
        e = (u - K["x"][idx].double()) ** 2 + (w - K["y"][idx].double()) ** 2
        ok &= e <= 5.991 * torch.from_numpy(SIGMA2).cuda().double()[K["octave"][idx].long()]
    ok = _winners(ok, h, q, j, len(R["x"]))
    depth[q] = torch.where(ok, X[:, 2], torch.full_like(D, -1.0))
    xyz[q] = torch.where(ok[:, None], X, torch.zeros_like(X))
    return depth, xyz


RING = [(0, -3), (1, -3), (2, -2), (3, -1), (3, 0), (3, 1), (2, 2), (1, 3), (0, 3), (-1, 3), (-2, 2), (-3, 1), (-3, 0),
        (-3, -1), (-2, -2), (-1, -3)]


def _exact_orb(case, seed):
    """(x, y, angle) of every corner, in 64 bits, zeros beyond their number."""
    data, lay = _orb_pyramid(case, seed)
    x, y, ang = [torch.zeros(65536, dtype=torch.float64, device="cuda") for _ in range(3)]
    at = 0
    dd = torch.arange(-15, 16, device="cuda")
    disc = (dd[:, None] ** 2 + dd ** 2 <= 225).long()
    for l in range(LEVELS):
        w, h = lay.width[l], lay.height[l]
        img = data[lay.offset[l]:lay.offset[l] + w * h].view(h, w).int()
        if w <= 38 or h <= 38:
            continue
        sc = torch.zeros((h, w), dtype=torch.int32, device="cuda")
        c = img[3:-3, 3:-3]
        e = torch.stack([img[3 + dy:h - 3 + dy, 3 + dx:w - 3 + dx] - c for dx, dy in RING])
        s = torch.full_like(c, -256)
        for k in range(16):
            arc = e[[(k + i) % 16 for i in range(9)]]
            s = torch.maximum(s, torch.maximum(arc.amin(0), -arc.amax(0)))
        s = s - 1
        sc[3:-3, 3:-3] = torch.where(s >= 20, s, torch.zeros_like(s))
        win = torch.zeros_like(sc)
        win[19:h - 19, 19:w - 19] = 1
        sc = sc * win
        keep = sc[1:-1, 1:-1] > 0
        for dy in (-1, 0, 1):
            for dx in (-1, 0, 1):
                if dx or dy:
                    keep &= sc[1:-1, 1:-1] > sc[1 + dy:h - 1 + dy, 1 + dx:w - 1 + dx]
        p = keep.nonzero() + 1
        p = p[:max(0, 65536 - at)]
        n = len(p)
        if not n:
            continue
        win = img[(p[:, 0, None, None] + dd[:, None]), (p[:, 1, None, None] + dd)].long() * disc
        m10, m01 = (win * dd).sum((1, 2)).double(), (win * dd[:, None]).sum((1, 2)).double()
        a = torch.atan2(m01, m10) * (180.0 / math.pi)
        x[at:at + n], y[at:at + n] = p[:, 1].double() * float(SF[l]), p[:, 0].double() * float(SF[l])
        ang[at:at + n] = torch.where(a < 0, a + 360.0, a)
        at += n
    return x, y, ang


def _exact_edit(case, seed):
    mp, ins, rem = _edit_inputs(case, seed)
    n, m = case["map"], len(rem)
    gone = np.zeros(n, bool)
    gone[rem] = True
    n1 = n - m
    holes, src = np.nonzero(gone[:n1])[0], n1 + np.nonzero(~gone[n1:])[0]
    out = {}
    for k, v in mp.items():
        if k != "order":
            v = v.double() if v.is_floating_point() else v
            v[torch.from_numpy(holes).cuda()] = v[torch.from_numpy(src).cuda()]
            v[n1:] = ins[k].to(v.dtype)
            out[k] = v if v.is_floating_point() else None
    return out


def exact(case, seed):
    kind = case["kind"]
    if kind in ("search", "last", "pyramid"):
        return None                                        # whole numbers only
    if kind == "orb":
        x, y, ang = _exact_orb(case, seed)
        return {"x": x, "y": y, "angle": ang}
    if kind == "edit":
        return _exact_edit(case, seed)
    frames = _frames(case, seed)
    lay, total = _layout()
    ur, depth, xyz = [], [], []
    for f in frames:
        n = len(f["left"]["x"])
        zero = torch.zeros(n, dtype=torch.float64, device="cuda")
        if f["kind"] == "pinhole":
            build = _built_pyramid if kind == "batch" and case["images"] else _pyramid
            a, b = _exact_pinhole(f, [build(im, lay, total) for im in f["images"]])
            ur.append(a)
            depth.append(b)
            xyz.append(torch.zeros((n, 3), dtype=torch.float64, device="cuda"))
        else:
            b, c = _exact_fisheye(f)
            ur.append(zero)
            depth.append(b)
            xyz.append(c)
    out = {"depth": torch.cat(depth)}
    if any(f["kind"] == "pinhole" for f in frames):
        out["u_right"] = torch.cat(ur)
    if any(f["kind"] == "fisheye" for f in frames):
        out["xyz"] = torch.cat(xyz)
    return out

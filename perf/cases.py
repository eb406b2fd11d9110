"""Performance cases: what a user of this rasterizer has it do, through the public entry points.

Clouds are seeded on the GPU with the distributions of ``paper_1908_02681_amd.gen``: spheres (random
order), a LIDAR-like terrain in Morton order or shuffled, and the contention cloud (dense terrain plus
dense spheres).  Points, framebuffers, images and workspaces stay resident between passes, as a viewer
or a server keeps them; every pass renders a whole frame from them and leaves the framebuffers cleared
for the next.

Kinds of a case:
  frame   one view through rasterize_atomicmin / rasterize_hq_splat (path "direct"), rasterize_sorted
          (path "sorted") or rasterize_points (point sizes above one pixel, "size" > 1);
  batch   many views of one resident cloud in one captured submission (Batch);
  serve   a burst of mixed requests through the render server (Server), submitted and drained.
"""
import math
import random

import numpy as np
import torch

from paper_1908_02681_amd import gen, rz

SIZES = [(256, 256), (640, 360), (640, 480), (1024, 768), (1280, 720), (1920, 1080), (2560, 1440)]
BATCH_SIZES = [(256, 256), (640, 480), (1280, 720), (1920, 1080)]
SERVE_CLOUDS = [1_000_000, 5_000_000, 20_000_000, 50_000_000]

# Sub-ranges of the paper's section 2.1: nanometres to 10 m, micrometres to 10 km, millimetres beyond.
PIECEWISE = ((0.0, 1e9), (10.0, 1e6), (10000.0, 1e3))


def _frame(name, cloud, n, order, w, h, hq, path="direct", size=1, depth="linear", off=0, eps=100,
           elev=45, dist=1000):
    c = {"kind": "frame", "cloud": cloud, "n": n, "order": order, "w": w, "h": h, "hq": hq,
         "path": path, "size": size, "depth": depth, "off": off, "eps": eps, "elev": elev,
         "dist": dist}
    return c if name is None else dict(c, name=name)


def listed():
    return [
        # a small object in an interactive viewer: latency and launches
        _frame("spheres100k_min_640x480", "spheres", 100_000, "shuffled", 640, 480, False),
        # the 1M-point sphere scene at 1024x768, splatted
        _frame("spheres1m_hq_1024x768", "spheres", 1_000_000, "shuffled", 1024, 768, True),
        # the benchmark scene (50M LIDAR-like points in Morton order, 1080p), both methods
        _frame("terrain50m_min_1080p", "terrain", 50_000_000, "morton", 1920, 1080, False),
        _frame("terrain50m_hq_1080p", "terrain", 50_000_000, "morton", 1920, 1080, True),
        # the contention scene, 300M points, splatted at 1440p: the largest single frame
        _frame("stress300m_hq_1440p", "stress", 300_000_000, "morton", 2560, 1440, True),
        # one device's share (an eighth, a ragged slice of the planes) of the benchmark scene under the
        # paper's piecewise depth map
        _frame("share6m_piecewise_min_1080p", "terrain", 6_250_003, "morton", 1920, 1080, False,
               depth="piecewise", off=3),
        # scans delivered in no particular order, through the screen-sorted path
        _frame("shuffled50m_sorted_hq_1080p", "terrain", 50_000_000, "shuffled", 1920, 1080, True,
               path="sorted"),
        _frame("shuffled20m_sorted_min_1440p", "terrain", 20_000_000, "shuffled", 2560, 1440, False,
               path="sorted"),
        # points larger than a pixel: sparse clouds closed up, and the 24-bit depth buffer for
        # comparison of precision
        _frame("terrain50m_size3_hq_1080p", "terrain", 50_000_000, "morton", 1920, 1080, True, size=3),
        _frame("terrain20m_size2_gl24_720p", "terrain", 20_000_001, "morton", 1280, 720, False, size=2,
               depth="gl24"),
        # 64 orbit views of a resident 100M-point cloud, half of them splatted, one captured graph
        {"name": "batch64_100m", "kind": "batch", "cloud": "terrain", "n": 100_000_000,
         "order": "morton", "views": 64, "trace": 3},
        # a burst of requests of mixed cloud, resolution and method through the render server
        {"name": "serve32_mixed", "kind": "serve", "requests": 32, "trace": 4},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choices(["direct", "sorted", "points", "batch", "serve"], [8, 4, 4, 2, 1])[0]
    if kind == "batch":
        n = _log(rng, 1_000_000, 100_000_000)
        return {"kind": "batch", "cloud": "terrain", "n": n, "order": "morton",
                "views": min(rng.randint(3, 64), 3_200_000_000 // n), "trace": rng.randrange(1 << 20)}
    if kind == "serve":
        return {"kind": "serve", "requests": rng.randint(4, 32), "trace": rng.randrange(1 << 20)}
    w, h = rng.choice(SIZES)
    if rng.random() < 0.5:   # windows of any size
        w, h = _log(rng, 200, 2560), _log(rng, 150, 1440)
    hq = rng.random() < 0.5
    depth = rng.choice(["linear", "linear", "scale", "piecewise"])
    eps = rng.choice([100, 100, 50, 200])
    off = rng.choice([0, 0, 0, rng.randint(1, 3)])
    elev, dist = rng.randint(20, 60), rng.randint(600, 1200)
    if kind == "sorted":
        n = _log(rng, 200_000, 60_000_000)
        cloud = rng.choice(["terrain", "spheres"])
        return _frame(None, cloud, n, "shuffled", w, h, hq, "sorted", 1, depth, off, eps, elev, dist)
    if kind == "points":
        n = _log(rng, 100_000, 50_000_000)
        if not hq:
            depth = rng.choice([depth, "gl24", "f32rev"])
        return _frame(None, "terrain", n, "morton", w, h, hq, "direct", rng.randint(2, 5), depth, off,
                      eps, elev, dist)
    if not hq:
        depth = rng.choice([depth, depth, "gl24", "f32rev"])
    cloud = rng.choice(["terrain", "terrain", "stress", "spheres"])
    n = _log(rng, 20_000, 4_000_000) if cloud == "spheres" else _log(rng, 200_000, 200_000_000)
    order = "shuffled" if cloud == "spheres" else "morton"
    return _frame(None, cloud, n, order, w, h, hq, "direct", 1, depth, off, eps, elev, dist)


# ---- clouds ----------------------------------------------------------------

def _gen(seed, salt):
    g = torch.Generator(device="cuda")
    g.manual_seed((seed * 1000003 + salt) % (1 << 62))
    return g


def _rgb(r, g, b):
    return r.int() | (g.int() << 8) | (b.int() << 16)


def _unit(n, g):
    d = torch.randn(3, n, generator=g, device="cuda")
    return d / d.norm(dim=0).clamp_min_(1e-20)


def _spheres(n, seed):
    """Points on the surfaces of 8 spheres, uniform colours, random order."""
    g, rng = _gen(seed, 1), np.random.default_rng([seed, 1])
    centre = torch.tensor(rng.uniform(0, 1, (3, 8)), dtype=torch.float32, device="cuda")
    rad = torch.tensor(rng.uniform(0.1, 0.5, 8), dtype=torch.float32, device="cuda")
    share = torch.cumsum(rad * rad, 0) / (rad * rad).sum()
    which = torch.searchsorted(share, torch.rand(n, generator=g, device="cuda")).clamp_max_(7)
    p = centre[:, which] + rad[which] * _unit(n, g)
    c = torch.randint(0, 256, (3, n), generator=g, device="cuda", dtype=torch.uint8)
    return rz.Points(p[0].contiguous(), p[1].contiguous(), p[2].contiguous(), _rgb(*c))


def _height(x, y, seed):
    """Six octaves of value noise over the square kilometre, amplitude 50 m."""
    z, amp, total = torch.zeros_like(x), 1.0, 0.0
    for k in range(6):
        lam = 200.0 / 2 ** k
        m = int(math.ceil(1000.0 / lam)) + 2
        lat = torch.tensor(np.random.default_rng([seed, 2, k]).uniform(-1, 1, m * m),
                           dtype=torch.float32, device="cuda")
        u, v = x / lam, y / lam
        iu, iv = u.int().clamp_(0, m - 2), v.int().clamp_(0, m - 2)
        tu, tv = u - iu, v - iv
        tu, tv = tu * tu * (3 - 2 * tu), tv * tv * (3 - 2 * tv)
        i = iv * m + iu
        lo = torch.lerp(lat[i], lat[i + 1], tu)
        z += amp * torch.lerp(lo, torch.lerp(lat[i + m], lat[i + m + 1], tu), tv)
        total += amp
        amp *= 0.5
    return z * (50.0 / total)


def _even_bits(v):
    v = v & 0x55555555
    for s, m in ((1, 0x33333333), (2, 0x0F0F0F0F), (4, 0x00FF00FF), (8, 0x0000FFFF)):
        v = (v | (v >> s)) & m
    return v


_RAMP = torch.tensor([[40, 90, 30], [110, 160, 60], [140, 110, 70], [225, 222, 212]],
                     dtype=torch.float32)


def _terrain(n, seed):
    """A jittered grid over the square kilometre in Morton order, coloured by height."""
    g = _gen(seed, 2)
    side = max(1, math.ceil(math.sqrt(n)))
    bits = max(1, math.ceil(math.log2(side)))
    step = 1000.0 / side
    out = [torch.empty(n, device="cuda") for _ in range(3)]
    out.append(torch.empty(n, dtype=torch.int32, device="cuda"))
    have, piece = 0, 1 << 24
    ramp = _RAMP.cuda()
    for code0 in range(0, 1 << (2 * bits), piece):
        code = torch.arange(code0, min(code0 + piece, 1 << (2 * bits)), dtype=torch.int32,
                            device="cuda")
        i, j = _even_bits(code), _even_bits(code >> 1)
        inside = (i < side) & (j < side)
        i, j = i[inside][:n - have], j[inside][:n - have]
        m = i.numel()
        if m:
            jit = torch.randn(3, m, generator=g, device="cuda") * (0.02 * step)
            cx, cy = (i + 0.5) * step, (j + 0.5) * step
            z = _height(cx, cy, seed)
            t = ((z + 50.0) / 100.0).clamp_(0, 1) * 3
            k = t.int().clamp_max_(2)
            col = torch.lerp(ramp[k], ramp[k + 1], (t - k)[:, None])
            col = col + torch.randint(-12, 13, (m, 3), generator=g, device="cuda")
            col = col.round_().clamp_(0, 255)
            e = have + m
            out[0][have:e] = cx + jit[0]
            out[1][have:e] = cy + jit[1]
            out[2][have:e] = z + jit[2]
            out[3][have:e] = _rgb(col[:, 0], col[:, 1], col[:, 2])
            have = e
        if have == n:
            break
    return rz.Points(*out)


def _spread3(v):
    for s, m in ((32, 0x1F00000000FFFF), (16, 0x1F0000FF0000FF), (8, 0x100F00F00F00F00F),
                 (4, 0x10C30C30C30C30C3), (2, 0x1249249249249249)):
        v = (v | (v << s)) & m
    return v


def _stress(n, seed):
    """Five sixths terrain, one sixth in 20 dense spheres on it, each in 3D Morton order."""
    per = n // 120
    t = _terrain(n - 20 * per, seed)
    g, rng = _gen(seed, 3), np.random.default_rng([seed, 3])
    cx, cy, r = rng.uniform(100, 900, 20), rng.uniform(100, 900, 20), rng.uniform(10, 40, 20)
    ground = _height(torch.tensor(cx, dtype=torch.float32, device="cuda"),
                     torch.tensor(cy, dtype=torch.float32, device="cuda"), seed).tolist()
    parts = [[t.x], [t.y], [t.z], [t.rgb]]
    for b in range(20 if per else 0):
        d = _unit(per, g)
        q = ((d + 1) * (0.5 * ((1 << 21) - 1))).long()
        o = torch.argsort(_spread3(q[0]) | (_spread3(q[1]) << 1) | (_spread3(q[2]) << 2))
        c = torch.randint(0, 256, (3, per), generator=g, device="cuda", dtype=torch.uint8)
        parts[0].append((d[0] * r[b] + cx[b])[o])
        parts[1].append((d[1] * r[b] + cy[b])[o])
        parts[2].append((d[2] * r[b] + (ground[b] + 0.5 * r[b]))[o])
        parts[3].append(_rgb(*c)[o])
    return rz.Points(*[torch.cat(p) for p in parts])


def _cloud(kind, n, order, seed, off=0):
    """off > 0: a slice of larger planes that starts `off` elements in."""
    make = {"spheres": _spheres, "terrain": _terrain, "stress": _stress}[kind]
    p = make(n + off, seed)
    planes = [p.x, p.y, p.z, p.rgb]
    if order == "shuffled" and kind != "spheres":
        perm = torch.randperm(n + off, generator=_gen(seed, 4), device="cuda")
        planes = [a[perm] for a in planes]
    return rz.Points(*[a[off:] for a in planes])


def _depth(kind):
    if kind == "scale":
        return rz.depth_struct(rz.DEPTH_SCALE, 1000.0)
    if kind == "piecewise":
        return rz.depth_struct(rz.DEPTH_PIECEWISE, PIECEWISE)
    return rz.depth_struct({"linear": rz.DEPTH_LINEAR, "gl24": rz.DEPTH_GL24,
                            "f32rev": rz.DEPTH_F32REV}[kind])


# ---- cases -----------------------------------------------------------------

def _requests(case):
    """The (cloud, width, height, splat) of a burst's requests."""
    rng = random.Random(case["trace"])
    return [(rng.randrange(len(SERVE_CLOUDS)), *rng.choice(gen.SERVE_SIZES), rng.random() < 0.5)
            for _ in range(case["requests"])]


def _batch_views(case):
    """The (width, height, splat) of a batch's views."""
    rng = random.Random(case["trace"])
    return [(*rng.choice(BATCH_SIZES), rng.random() < 0.5) for _ in range(case["views"])]


def prepare(case, seed):
    if case["kind"] == "batch":
        pts = _cloud(case["cloud"], case["n"], case["order"], seed)
        spec = _batch_views(case)
        views = [gen.orbit_views(1, seed * 4096 + i, [(w, h)])[0] for i, (w, h, _) in enumerate(spec)]
        # the shape that the batch autotuner settles on for this kind of cloud, kept by the program
        b = rz.Batch(pts, views, [rz.RZ_MODE_HQ if hq else rz.RZ_MODE_ATOMICMIN for *_, hq in spec],
                     views_per_group=8, launch=(256, 4, 1, 0, 3), use_graph=True)
        return {"case": case, "batch": b}
    if case["kind"] == "serve":
        spec = _requests(case)
        clouds = [_cloud("spheres" if i == 0 else "terrain", n, "morton", seed * 8 + i)
                  for i, n in enumerate(SERVE_CLOUDS)]
        srv = rz.Server(1 << 30, streams=4, work_cap=100_000_000)
        ids = [srv.add_cloud(c) for c in clouds]
        reqs = []
        for i, (c, w, h, hq) in enumerate(spec):
            if c == 0:
                v = gen.orbit_views(1, seed * 4096 + i, [(w, h)], extent=1.0, rmin=1.5, rmax=3.0,
                                    elev=(-60.0, 60.0), near=0.01, far=10.0)[0]
            else:
                v = gen.orbit_views(1, seed * 4096 + i, [(w, h)])[0]
            img = torch.zeros(w * h, dtype=torch.int32, device="cuda")
            reqs.append((ids[c], v, rz.RZ_MODE_HQ if hq else rz.RZ_MODE_ATOMICMIN, img))
        return {"case": case, "server": srv, "requests": reqs}
    pts = _cloud(case["cloud"], case["n"], case["order"], seed, case["off"])
    w, h = case["w"], case["h"]
    if case["cloud"] == "spheres":
        view = gen.make_view((0.5, 0.5, 2.5), (0.5, 0.5, 0.5), (0, 1, 0), 60.0, w, h, 0.01, 10.0)
    else:
        view = gen.terrain_view(w, h, distance=case["dist"], elevation_deg=case["elev"])
    fb, acc = rz.new_framebuffer(view, 0x102030, hq=case["hq"])
    s = {"case": case, "points": pts, "view": view, "depth": _depth(case["depth"]), "fb": fb,
         "acc": acc, "img": torch.empty(w * h, dtype=torch.int32, device="cuda")}
    if case["hq"]:
        s["status"] = torch.zeros(1, dtype=torch.int32, device="cuda")
    if case["path"] == "sorted":
        s["workspace"] = rz.new_workspace(pts.n, w, h)
    return s


def run(s):
    case = s["case"]
    if case["kind"] == "batch":
        s["batch"].run()
        return s["batch"].imgs
    if case["kind"] == "serve":
        for c, v, mode, img in s["requests"]:
            s["server"].submit(c, v, mode, img)
        s["server"].drain()
        return [r[3] for r in s["requests"]]
    kw = {"depth": s["depth"], "background": 0x102030, "fb": s["fb"], "img": s["img"]}
    if case["hq"]:
        kw.update(acc=s["acc"], status=s["status"], eps=(1, case["eps"]))
    if case["path"] == "sorted":
        rz.rasterize_sorted(s["points"], s["view"], hq=case["hq"], workspace=s["workspace"], **kw)
    elif case["size"] > 1:
        rz.rasterize_points(s["points"], s["view"], hq=case["hq"], point_size=case["size"], **kw)
    elif case["hq"]:
        rz.rasterize_hq_splat(s["points"], s["view"], **kw)
    else:
        rz.rasterize_atomicmin(s["points"], s["view"], **kw)
    out = [s["img"], s["fb"]]
    return out + [s["acc"], s["status"]] if case["hq"] else out


def work(case):
    """Each point read once (16 bytes) and each pixel's colour written once.  Per point and view about
    50 operations (projection, depth, key), 25 more for a splat's window and sums."""
    if case["kind"] == "batch":
        v = _batch_views(case)
        return {"bytes": 16 * case["n"] + 4 * sum(w * h for w, h, _ in v),
                "flops": case["n"] * sum(75 if hq else 50 for *_, hq in v)}
    if case["kind"] == "serve":
        r = _requests(case)
        return {"bytes": sum(16 * SERVE_CLOUDS[c] + 4 * w * h for c, w, h, _ in r),
                "flops": sum(SERVE_CLOUDS[c] * (75 if hq else 50) for c, *_, hq in r)}
    n, px = case["n"], case["w"] * case["h"]
    k2 = case["size"] ** 2
    return {"bytes": 16 * n + 4 * px, "flops": n * (50 + (25 * k2 if case["hq"] else 2 * (k2 - 1)))}


def exact(case, seed):
    """Images, keys and sums are whole numbers (packed words), fixed bit for bit by the interface."""
    return None

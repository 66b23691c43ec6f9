"""The measured workloads: what a user's program has this rasterizer do, through
its public entry points, from one small frame to a sixteen-camera batch.

Kinds (``case["kind"]``):
  frame       Renderer.render: projection, ordering and raster of one camera
  project     project: projection and colour alone
  bin         Renderer.bin: the depth-binned ordering alone
  raster      Renderer.rasterize over a binned stream (keeping the final
              transmittance, as a training forward does)
  raster_bwd  Renderer.rasterize_backward from the forward's saved state
  train       render_differentiable, a mean squared error and its gradients
              with respect to every Gaussian parameter
  batch       BatchRenderer over several cameras, eagerly or replayed from its
              HIP graph

Inputs are drawn on the GPU from the seed alone. Two scene structures, those of
the synthetic workloads: ``box`` (means uniform in a box, dense at the
resolutions used here: long per-tile ranges everywhere) and ``surface`` (means on
random spheres and planes, strongly uneven tiles: most empty, some with
thousands of entries). ``shuffled`` stores the surface Gaussians in random order
(as after densification); otherwise one primitive follows another.

``exact`` evaluates the image model in binary64 with plain torch: the
projection, the compositing in (binary32 depth, id) order over per-tile lists,
and its gradients (the projection's by autograd).
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2609_03613_amd as tg

KEYS = ("means", "log_scales", "quats", "logits", "sh")


# ---------------------------------------------------------------------------
# cases
# ---------------------------------------------------------------------------

def _case(kind, scene, n, width, height, degree, tile=16, bins=64, sub=0, shuffled=False, **kw):
    return dict(kind=kind, scene=scene, n=n, width=width, height=height, degree=degree, tile=tile, bins=bins, sub=sub, shuffled=shuffled, **kw)


def listed():
    return [
        # a thumbnail or an interactive preview: a few thousand Gaussians, all latency and launches
        dict(_case("frame", "box", 2000, 128, 128, 0), name="frame_2k_128x128"),
        # a low-resolution view of a full scene: few tiles, each with thousands of entries
        dict(_case("frame", "surface", 1_000_000, 640, 360, 3), name="frame_1m_640x360"),
        # the ordinary frame: a trained-model-sized scene (SH degree 3) at 1080p
        dict(_case("frame", "surface", 1_000_000, 1920, 1080, 3), name="frame_1m_1920x1080"),
        # the largest single frame: 6M Gaussians at 4K
        dict(_case("frame", "surface", 6_000_000, 3840, 2160, 3), name="frame_6m_3840x2160"),
        # the projection layer alone, as a program that keeps splats between calls has it
        dict(_case("project", "surface", 1_000_000, 1920, 1080, 3), name="project_1m_sh3"),
        # the ordering layer alone at scale: 10M Gaussians in random order, segments of thousands of entries
        dict(_case("bin", "surface", 10_000_000, 1920, 1080, 0, shuffled=True), name="bin_10m_1920x1080"),
        # the raster layer on a uniformly dense scene (the training forward's)
        dict(_case("raster", "box", 500_000, 1297, 840, 0), name="raster_500k_1297x840"),
        # its backward with the tile size and bins that the autotuner picks on such a scene
        dict(_case("raster_bwd", "box", 500_000, 1297, 840, 0, 32, 128, 2), name="raster_bwd_500k_t32"),
        # an optimisation step on a small crop with ragged tiles: launches and latency
        dict(_case("train", "box", 20_000, 333, 257, 3), name="train_20k_333x257"),
        # the ordinary optimisation step
        dict(_case("train", "box", 500_000, 1297, 840, 3), name="train_500k_1297x840"),
        # a few cameras rendered eagerly, with the default options
        dict(_case("batch", "box", 60_000, 640, 360, 0, views=4, span=2.0, graph=False), name="batch_4_views_60k"),
        # serving many cameras of one large scene from a captured graph, with tuned options
        dict(_case("batch", "box", 3_000_000, 640, 360, 0, 32, 128, 2, views=16, span=4.0, graph=True),
             name="batch_16_views_3m"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("frame", "frame", "frame", "project", "bin", "raster", "raster_bwd", "train", "train", "batch"))
    degree = rng.choice((0, 1, 2, 3, 3))
    shuffled = rng.random() < 0.5
    # 16-pixel tiles with 64 bins are the default; the others are what the autotuner chooses from
    tile, bins, sub = rng.choice(((16, 64, 0), (16, 64, 0), (16, 64, 0), (16, 128, 4), (8, 32, 0), (32, 128, 2)))
    if kind == "batch":
        n = _log_int(rng, 20_000, 1_000_000)
        views = rng.randint(2, 12)
        return _case(kind, "box", n, rng.randint(200, 640), rng.randint(150, 360), 0, *rng.choice(((16, 64, 0), (32, 128, 2))),
                     views=views, span=rng.choice((1.0, 2.0, 3.0)), graph=rng.random() < 0.5)
    width = _log_int(rng, 128, 3840)
    height = max(96, min(2160, int(width * rng.uniform(0.5, 1.0))))
    if kind == "frame":
        scene = rng.choice(("surface", "surface", "box"))
        n = _log_int(rng, 2000, 4_000_000 if scene == "surface" else 500_000)
        return _case(kind, scene, n, width, height, degree, tile, bins, sub, shuffled)
    if kind == "project":
        return _case(kind, rng.choice(("surface", "box")), _log_int(rng, 5000, 4_000_000), width, height, degree, tile, bins, sub, shuffled)
    if kind == "bin":
        width, height = min(width, 1920), min(height, 1080)
        return _case(kind, "surface", _log_int(rng, 20_000, 10_000_000), width, height, 0, tile, bins, sub, shuffled)
    width = _log_int(rng, 160, 1600)
    height = max(96, min(1080, int(width * rng.uniform(0.5, 1.0))))
    n = _log_int(rng, 5000, 500_000)
    scene = rng.choice(("box", "box", "surface"))
    if kind == "train":
        return _case(kind, scene, n, width, height, degree, tile, bins, sub, shuffled)
    return _case(kind, scene, n, width, height, 0, tile, bins, sub, shuffled)


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _uniform(gen, lo, hi, *shape):
    return torch.rand(*shape, generator=gen, device="cuda") * (hi - lo) + lo


def _normal(gen, mean, std, *shape):
    return torch.randn(*shape, generator=gen, device="cuda") * std + mean


def _gaussians(case, seed):
    """The scene's Gaussians as float32 CUDA tensors in the library's layout."""
    gen, n, degree = _gen(seed), case["n"], case["degree"]
    if case["scene"] == "box":
        u = torch.rand(n, 3, generator=gen, device="cuda")
        means = u * torch.tensor([2.0, 2.0, 4.0], device="cuda") + torch.tensor([-1.0, -1.0, 2.0], device="cuda")
        log_scales = _normal(gen, -4.0, 0.5, n, 3)
        logit_std = 1.5
    else:
        prims = 64
        k = torch.arange(n, device="cuda")
        k = k % prims if case["shuffled"] else k * prims // n
        centres = _uniform(gen, -4.0, 4.0, prims, 3)
        radii, sides = _uniform(gen, 0.5, 2.0, prims), _uniform(gen, 1.0, 4.0, prims)
        frame = torch.linalg.qr(torch.randn(prims, 3, 3, generator=gen, device="cuda"))[0]
        d = torch.nn.functional.normalize(torch.randn(n, 3, generator=gen, device="cuda"), dim=1)
        uv = torch.rand(n, 2, generator=gen, device="cuda") - 0.5
        off = _normal(gen, 0.0, 0.01, n, 1)
        sphere = d * (radii[k][:, None] + off)
        f = frame[k]
        plane = sides[k][:, None] * (uv[:, :1] * f[:, 0] + uv[:, 1:] * f[:, 1]) + off * f[:, 2]
        means = (centres[k] + torch.where((k % 2 == 0)[:, None], sphere, plane)).clamp(-5.0, 5.0)
        log_scales = _normal(gen, -4.5, 0.7, n, 3)
        logit_std = 2.0
    quats = torch.nn.functional.normalize(torch.randn(n, 4, generator=gen, device="cuda"), dim=1)
    logits = _normal(gen, 0.0, logit_std, n)
    if degree == 0:
        sh = _uniform(gen, -math.sqrt(math.pi), math.sqrt(math.pi), n, 1, 3)
    else:
        sh = _normal(gen, 0.0, 0.2, n, (degree + 1) ** 2, 3)
    g = {"means": means, "log_scales": log_scales, "quats": quats, "logits": logits, "sh": sh}
    g = {k: v.float().contiguous() for k, v in g.items()}
    g["sh_degree"] = degree
    return g


def _camera(case):
    """The box is seen from the origin at f = width, the surfaces from z = -15 at
    f = 1100 for 1920 pixels of width."""
    w, h = case["width"], case["height"]
    f, z = (float(w), 0.0) if case["scene"] == "box" else (1100.0 * w / 1920.0, 15.0)
    return {"R": np.eye(3), "t": np.array([0.0, 0.0, z]), "fx": f, "fy": f, "cx": w / 2.0, "cy": h / 2.0, "width": w,
            "height": h, "znear": 0.01, "zfar": 1e10}


def _ring(case):
    """The batch's cameras: a ring of radius 5 around the box, looking at its
    centre, image sizes spread over 1 .. span times the base size."""
    cams, nv = [], case["views"]
    for v in range(nv):
        th = 2.0 * math.pi * v / nv
        pos, centre = np.array([5.0 * math.sin(th), 0.0, 4.0 - 5.0 * math.cos(th)]), np.array([0.0, 0.0, 4.0])
        f = (centre - pos) / np.linalg.norm(centre - pos)
        y = np.array([0.0, 1.0, 0.0])
        R = np.stack([np.cross(y, f), y, f])
        s = 1.0 + (case["span"] - 1.0) * ((v * 7) % nv) / max(nv - 1, 1)
        w, h = int(round(case["width"] * s)), int(round(case["height"] * s))
        cams.append({"R": R, "t": -R @ pos, "fx": float(w), "fy": float(w), "cx": w / 2.0, "cy": h / 2.0, "width": w,
                     "height": h, "znear": 0.01, "zfar": 1e10})
    return cams


def _params(case):
    return tg.Params(tile_size=case["tile"], num_bins=case["bins"], sub_bins=case["sub"])


def _splats(case, seed):
    """Projected splats and info lines of the scene (the binary64 projection
    below, rounded to the library's layout), for the single layers."""
    g, cam = _gaussians(case, seed), _camera(case)
    P = _project64(_doubles(g), case["degree"], cam, case["tile"])
    return _pack_splats(P), P["info"]


def _target(case, seed):
    return torch.rand(case["height"], case["width"], 3, generator=_gen(seed + 7_000_003), device="cuda")


def prepare(case, seed):
    kind = case["kind"]
    if kind == "batch":
        br = tg.BatchRenderer(_ring(case), [_params(case) for _ in range(case["views"])])
        g = _gaussians(case, seed)
        if case["graph"]:
            br.capture(g)
        else:
            br.frame(g, sync=True)  # sizes the entry buffers, as the class asks for
        return {"kind": kind, "br": br, "g": g, "graph": case["graph"]}
    r = tg.Renderer(_camera(case), _params(case))
    s = {"kind": kind, "r": r}
    if kind in ("frame", "project"):
        s["g"] = _gaussians(case, seed)
    elif kind == "train":
        s["g"] = _gaussians(case, seed)
        for k in KEYS:
            s["g"][k].requires_grad_(True)
        s["target"] = _target(case, seed)
    else:
        s["splats"], s["info"] = _splats(case, seed)
        if kind == "bin":
            # entry buffers of a stated capacity, above the entries of these scenes; their unused end stays zero
            r.bin(s["splats"], s["info"], capacity=(12 if case["tile"] == 8 else 4) * case["n"]).pairs.zero_()
        else:
            s["binned"] = r.bin(s["splats"], s["info"])
        if kind == "raster_bwd":
            s["saved"] = r.rasterize(s["splats"], s["info"], s["binned"], trans=True)
            s["d_rgb"] = (s["saved"]["rgb"] - _target(case, seed)) * (2.0 / (3 * case["width"] * case["height"]))
    return s


def run(s):
    kind = s["kind"]
    if kind == "batch":
        return s["br"].replay() if s["graph"] else s["br"].frame(s["g"])
    r = s["r"]
    if kind == "frame":
        out = r.render(s["g"])
        return {k: out[k] for k in ("rgb", "alpha", "last")}
    if kind == "project":
        splats, info = tg.project(s["g"], r.cam, r.params)
        return {"splats": splats, "info": info}
    if kind == "bin":
        b = r.bin(s["splats"], s["info"])
        return {"pairs": b.pairs, "offsets": b.offsets, "zrange": b.zrange, "counters": b.counters}
    if kind == "raster":
        return r.rasterize(s["splats"], s["info"], s["binned"], trans=True)
    if kind == "raster_bwd":
        return {"d_splats": r.rasterize_backward(s["splats"], s["info"], s["binned"], s["d_rgb"], saved=s["saved"])}
    rgb, alpha = tg.render_differentiable(r, s["g"])
    loss = ((rgb - s["target"]) ** 2).mean()
    grads = torch.autograd.grad(loss, [s["g"][k] for k in KEYS])
    return {"rgb": rgb, "alpha": alpha, "loss": loss, "grads": dict(zip(KEYS, grads))}


def work(case):
    """Bytes: inputs read once, outputs written once. Operations: about 250 per
    projected Gaussian, and 15 per alpha-supported pixel test (45 in the
    backward) at the scenes' typical counts per pixel."""
    kind, n, px = case["kind"], case["n"], case["width"] * case["height"]
    gauss = 4 * n * (11 + 3 * (case["degree"] + 1) ** 2)
    tests = 13 if case["scene"] == "surface" else 25
    if kind == "batch":
        px = sum(c["width"] * c["height"] for c in _ring(case))
        return {"bytes": gauss + 20 * px, "flops": 250 * n * case["views"] + 15 * tests * px}
    if kind == "frame":
        return {"bytes": gauss + 20 * px, "flops": 250 * n + 15 * tests * px}
    if kind == "project":
        return {"bytes": gauss + 80 * n, "flops": 250 * n}
    entries = 2.3 * n if case["scene"] == "surface" else 12 * n
    if kind == "bin":
        return {"bytes": 16 * n + 8 * entries, "flops": 0}
    if kind == "raster":
        return {"bytes": 48 * n + 8 * entries + 24 * px, "flops": 15 * tests * px}
    if kind == "raster_bwd":
        return {"bytes": 48 * n + 8 * entries + 20 * px + 48 * n, "flops": 45 * tests * px}
    return {"bytes": 2 * gauss + 20 * px + 12 * px, "flops": 750 * n + 60 * tests * px}


# ---------------------------------------------------------------------------
# the same in binary64
# ---------------------------------------------------------------------------

def _doubles(g):
    return {k: g[k].detach().double() for k in KEYS}


def _sh64(d, degree):
    x, y, z = d.unbind(1)
    Y = [torch.full_like(x, 0.5 / math.sqrt(math.pi))]
    if degree > 0:
        c = math.sqrt(3.0 / (4.0 * math.pi))
        Y += [-c * y, c * z, -c * x]
    if degree > 1:
        c = 0.5 * math.sqrt(15.0 / math.pi)
        Y += [c * x * y, -c * y * z, 0.25 * math.sqrt(5.0 / math.pi) * (2 * z * z - x * x - y * y), -c * x * z,
              0.5 * c * (x * x - y * y)]
    if degree > 2:
        a, b, e = 0.25 * math.sqrt(35.0 / (2 * math.pi)), 0.5 * math.sqrt(105.0 / math.pi), 0.25 * math.sqrt(21.0 / (2 * math.pi))
        Y += [-a * y * (3 * x * x - y * y), b * x * y * z, -e * y * (4 * z * z - x * x - y * y),
              0.25 * math.sqrt(7.0 / math.pi) * z * (2 * z * z - 3 * x * x - 3 * y * y), -e * x * (4 * z * z - x * x - y * y),
              0.5 * b * z * (x * x - y * y), -a * x * (x * x - 3 * y * y)]
    return torch.stack(Y, 1)


def _project64(g, degree, cam, ts):
    """Screen mean, conic, opacity, colour, largest scale, visibility and the
    info line of every Gaussian (differentiable in g)."""
    R = torch.tensor(np.asarray(cam["R"]), dtype=torch.float64, device="cuda")
    t = torch.tensor(np.asarray(cam["t"]), dtype=torch.float64, device="cuda")
    m = g["means"]
    p = [R[i, 0] * m[:, 0] + R[i, 1] * m[:, 1] + R[i, 2] * m[:, 2] + t[i] for i in range(3)]
    z = p[2]
    w, h, fx, fy = cam["width"], cam["height"], cam["fx"], cam["fy"]
    front = (z > cam["znear"]) & (z < cam["zfar"])
    zs = torch.where(front, z, torch.ones_like(z))
    q = g["quats"] / g["quats"].norm(dim=1, keepdim=True)
    qw, qx, qy, qz = q.unbind(1)
    Rq = torch.stack([1 - 2 * (qy * qy + qz * qz), 2 * (qx * qy - qw * qz), 2 * (qx * qz + qw * qy),
                      2 * (qx * qy + qw * qz), 1 - 2 * (qx * qx + qz * qz), 2 * (qy * qz - qw * qx),
                      2 * (qx * qz - qw * qy), 2 * (qy * qz + qw * qx), 1 - 2 * (qx * qx + qy * qy)], 1).view(-1, 3, 3)
    s = torch.exp(g["log_scales"])
    M = [R[i, 0] * Rq[:, 0] + R[i, 1] * Rq[:, 1] + R[i, 2] * Rq[:, 2] for i in range(3)]
    gx, gy = 0.15 * w / fx, 0.15 * h / fy
    tx = zs * (p[0] / zs).clamp(-(cam["cx"] / fx + gx), (w - cam["cx"]) / fx + gx)
    ty = zs * (p[1] / zs).clamp(-(cam["cy"] / fy + gy), (h - cam["cy"]) / fy + gy)
    A = ((fx / zs)[:, None] * M[0] - (fx * tx / (zs * zs))[:, None] * M[2]) * s
    B = ((fy / zs)[:, None] * M[1] - (fy * ty / (zs * zs))[:, None] * M[2]) * s
    c00, c01, c11 = (A * A).sum(1) + 0.3, (A * B).sum(1), (B * B).sum(1) + 0.3
    det = c00 * c11 - c01 * c01
    mx, my = fx * p[0] / zs + cam["cx"], fy * p[1] / zs + cam["cy"]
    o = torch.sigmoid(g["logits"])
    campos = -(R.T @ t)
    d = m - campos
    Y = _sh64(d / d.norm(dim=1, keepdim=True), degree)
    rgb = (0.5 + (Y[:, :, None] * g["sh"]).sum(1)).clamp(min=0.0)
    with torch.no_grad():
        ok = front & (det > 0) & (o >= 1.0 / 255.0)
        tau = 2.0 * torch.log((255.0 * o).clamp(min=1.0))
        ex, ey = torch.sqrt(tau * c00) * (1 + 1e-4) + 1e-3, torch.sqrt(tau * c11) * (1 + 1e-4) + 1e-3
        nx, ny = -(-w // ts), -(-h // ts)
        x0, x1 = ((mx - ex) / ts).floor().clamp(0, nx), (((mx + ex) / ts).floor() + 1).clamp(0, nx)
        y0, y1 = ((my - ey) / ts).floor().clamp(0, ny), (((my + ey) / ts).floor() + 1).clamp(0, ny)
        ok = ok & (x1 > x0) & (y1 > y0)
        x0, x1, y0, y1 = (torch.where(ok, v, torch.zeros_like(v)).to(torch.int64) for v in (x0, x1, y0, y1))
        depth = torch.where(ok, z, torch.zeros_like(z)).float().view(torch.int32)
        info = torch.stack([depth, (x0 | (y0 << 16)).to(torch.int32), (x1 | (y1 << 16)).to(torch.int32),
                            ((x1 - x0) * (y1 - y0)).to(torch.int32)], 1).contiguous()
    return {"mean": torch.stack([mx, my], 1), "conic": torch.stack([c11 / det, -c01 / det, c00 / det], 1), "o": o, "rgb": rgb,
            "smax": s.max(1).values, "ok": ok, "info": info}


def _pack_splats(P, dtype=torch.float32):
    n = P["o"].shape[0]
    out = torch.zeros(n, 16, dtype=torch.float64, device="cuda")
    hi = P["mean"].float().double()
    out[:, 0:2], out[:, 2:4] = hi, P["mean"] - hi
    out[:, 4:7], out[:, 7], out[:, 8:11], out[:, 11] = P["conic"], P["o"], P["rgb"], P["smax"]
    out[~P["ok"]] = 0.0
    return out.to(dtype)


def _of_splats(splats, info):
    s = splats.double()
    return {"mean": s[:, 0:2] + s[:, 2:4], "conic": s[:, 4:7], "o": s[:, 7], "rgb": s[:, 8:11], "info": info}


def _entries(info, cam, ts):
    """Gaussian ids in (tile, depth, id) order, and each tile's range."""
    nx, ny = -(-cam["width"] // ts), -(-cam["height"] // ts)
    i = info.to(torch.int64)
    x0, y0, x1 = i[:, 1] & 0xFFFF, i[:, 1] >> 16, i[:, 2] & 0xFFFF
    gid = torch.repeat_interleave(torch.arange(len(i), device="cuda"), i[:, 3])
    first = torch.cumsum(i[:, 3], 0) - i[:, 3]
    j = torch.arange(len(gid), device="cuda") - first[gid]
    wd = (x1 - x0)[gid].clamp(min=1)
    tile = (y0[gid] + j // wd) * nx + x0[gid] + j % wd
    order = torch.sort((tile << 32) | i[:, 0][gid], stable=True).indices
    off = torch.zeros(nx * ny + 1, dtype=torch.int64, device="cuda")
    off[1:] = torch.cumsum(torch.bincount(tile, minlength=nx * ny), 0)
    return gid[order], off


class _Walk:
    """Every tile's entries front to back, all tiles in step; tiles leave when
    their range ends or all their pixels have stopped."""

    def __init__(self, P, cam, ts):
        self.cam, self.ts = cam, ts
        self.gid, off = _entries(P["info"], cam, ts)
        self.f = torch.cat([P["mean"], P["conic"], P["o"][:, None], P["rgb"]], 1)
        self.nx, self.ny = -(-cam["width"] // ts), -(-cam["height"] // ts)
        cnt = off[1:] - off[:-1]
        self.t = torch.argsort(cnt, descending=True)
        self.begin, self.cnt = off[:-1][self.t], cnt[self.t]
        l = torch.arange(ts * ts, device="cuda")
        self.x = ((self.t % self.nx) * ts)[:, None] + (l % ts)[None]
        self.y = ((self.t // self.nx) * ts)[:, None] + (l // ts)[None]

    def tiles(self, image):
        """[H, W, C] -> [tile, pixel, C] in the walk's tile order (0 outside)."""
        H, W = image.shape[:2]
        v = image[self.y.clamp(max=H - 1), self.x.clamp(max=W - 1)]
        return torch.where(((self.y < H) & (self.x < W))[..., None], v, torch.zeros_like(v))

    def image(self, v):
        H, W = self.cam["height"], self.cam["width"]
        out = torch.zeros(self.ny * self.ts, self.nx * self.ts, v.shape[-1], dtype=v.dtype, device="cuda")
        out[self.y, self.x] = v
        return out[:H, :W].contiguous()

    def forward(self, visit=None):
        """Colour [T, P, 3] without background and final transmittance [T, P];
        visit(tiles, ids, terms) is called at every step."""
        nt, pp = self.x.shape
        inside = (self.y < self.cam["height"]) & (self.x < self.cam["width"])
        C = torch.zeros(nt, pp, 3, dtype=torch.float64, device="cuda")
        T = torch.ones(nt, pp, dtype=torch.float64, device="cuda")
        cnt = self.cnt.tolist()
        act = torch.arange(sum(c > 0 for c in cnt), device="cuda")
        sub = None
        i = 0
        while i < (cnt[0] if cnt else 0):
            if i % 32 == 0:  # the tiles still walking
                if sub is not None:
                    C[act], T[act] = sub[0], sub[1]
                    act = act[sub[2].any(1) & (self.cnt[act] > i)]
                    live = sub[2][keep_of(sub[3], act)]
                else:
                    live = inside[act]
                if not len(act):
                    break
                px, py = self.x[act] + 0.5, self.y[act] + 0.5
                b, c = self.begin[act], self.cnt[act]
                sub = [C[act], T[act], live, act]
            has = i < c
            ids = self.gid[(b + i).clamp(max=len(self.gid) - 1)]
            e = self.f[ids]
            dx, dy = e[:, 0:1] - px, e[:, 1:2] - py
            qa, qb, qc = e[:, 2:3], e[:, 3:4], e[:, 4:5]
            G = torch.exp(-0.5 * (qa * dx * dx + 2 * qb * dx * dy + qc * dy * dy))
            araw = e[:, 5:6] * G
            alpha = araw.clamp(max=0.99)
            sup = sub[2] & (araw >= 1.0 / 255.0) & has[:, None]
            nxt = sub[1] * (1 - alpha)
            comp = sup & (nxt >= 1e-4)
            sub[2] = sub[2] & ~(sup & ~comp)
            wt = torch.where(comp, sub[1] * alpha, torch.zeros_like(alpha))
            sub[0] = sub[0] + wt[..., None] * e[:, None, 6:9]
            if visit is not None:
                visit(act, ids, e, dx, dy, G, araw, alpha, comp, sub[1], wt, sub[0])
            sub[1] = torch.where(comp, nxt, sub[1])
            i += 1
        if sub is not None and len(sub[3]):
            C[sub[3]], T[sub[3]] = sub[0], sub[1]
        return C, T

    def backward(self, d_rgb):
        """dL/d(mean, conic, opacity, rgb) [n, 9] for dL/d rgb [H, W, 3] (no
        background, no gradient on alpha)."""
        C, _ = self.forward()
        g = self.tiles(d_rgb.double())
        out = torch.zeros(self.f.shape[0], 9, dtype=torch.float64, device="cuda")

        def visit(act, ids, e, dx, dy, G, araw, alpha, comp, T, wt, acc):
            ga = g[act]
            behind = C[act] - acc
            da = (ga * (T[..., None] * e[:, None, 6:9] - behind / (1 - alpha)[..., None])).sum(2)
            da = torch.where(comp, da, torch.zeros_like(da))
            dn = torch.where(araw <= 0.99, da, torch.zeros_like(da))
            dq = -0.5 * dn * araw
            qa, qb, qc = e[:, 2:3], e[:, 3:4], e[:, 4:5]
            v = [(dq * 2 * (qa * dx + qb * dy)).sum(1), (dq * 2 * (qb * dx + qc * dy)).sum(1), (dq * dx * dx).sum(1),
                 (dq * 2 * dx * dy).sum(1), (dq * dy * dy).sum(1), (dn * G).sum(1)]
            out.index_add_(0, ids, torch.cat([torch.stack(v, 1), (ga * wt[..., None]).sum(1)], 1))

        self.forward(visit)
        return out


def keep_of(old, new):
    """Rows of ``old`` (ascending) that ``new``, a subset of it, holds."""
    return torch.searchsorted(old, new)


def exact(case, seed):
    kind = case["kind"]
    if kind == "batch":
        if case["n"] > 200_000:
            return None
        g = _doubles(_gaussians(case, seed))
        outs = []
        for cam in _ring(case):
            w = _Walk(_project64(g, case["degree"], cam, case["tile"]), cam, case["tile"])
            C, T = w.forward()
            outs.append({"rgb": w.image(C), "alpha": w.image((1 - T)[..., None])[..., 0], "last": None})
        return outs
    cam, ts = _camera(case), case["tile"]
    if kind in ("frame", "project", "train"):
        g = _doubles(_gaussians(case, seed))
        if kind == "train":
            for k in KEYS:
                g[k].requires_grad_(True)
        P = _project64(g, case["degree"], cam, ts)
        if kind == "project":
            return {"splats": _pack_splats(P, torch.float64), "info": None}
        Q = {k: v.detach() for k, v in P.items()}
    else:
        splats, info = _splats(case, seed)
        Q = _of_splats(splats, info)
    if kind == "bin":
        z = info[:, 0][info[:, 3] != 0].view(torch.float32).double()
        V, S = len(z), 8192
        if V > S:
            z = z[torch.arange(S, device="cuda") * V // S]
        z = z.sort().values
        lo, hi = z[int(math.floor(0.01 * (len(z) - 1)))].item(), z[int(math.ceil(0.99 * (len(z) - 1)))].item()
        pad = 0.05 * max(hi - lo, 1e-6)
        zr = torch.tensor([max(lo - pad, cam["znear"]), min(hi + pad, cam["zfar"])], dtype=torch.float64, device="cuda")
        return {"pairs": None, "offsets": None, "zrange": zr, "counters": None}
    w = _Walk(Q, cam, ts)
    if kind == "raster_bwd":
        C, _ = w.forward()
        d = torch.zeros(case["n"], 12, dtype=torch.float64, device="cuda")
        scale = 2.0 / (3 * case["width"] * case["height"])
        d[:, :9] = w.backward((w.image(C) - _target(case, seed)) * scale)
        return {"d_splats": d}
    C, T = w.forward()
    rgb, trans = w.image(C), w.image(T[..., None])[..., 0]
    if kind == "frame":
        return {"rgb": rgb, "alpha": 1 - trans, "last": None}
    if kind == "raster":
        return {"rgb": rgb, "alpha": 1 - trans, "last": None, "trans": trans}
    diff = rgb - _target(case, seed).double()
    d = w.backward(diff * (2.0 / diff.numel()))
    d = torch.where(P["ok"][:, None], d, torch.zeros_like(d))
    heads = [P["mean"], P["conic"], P["o"], P["rgb"]]
    grads = torch.autograd.grad(heads, [g[k] for k in KEYS], [d[:, 0:2], d[:, 2:5], d[:, 5], d[:, 6:9]])
    return {"rgb": rgb, "alpha": 1 - trans, "loss": (diff ** 2).mean(), "grads": dict(zip(KEYS, grads))}

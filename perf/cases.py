"""Work that a user of the rasterizer has it do, as measurable cases.

Every case is one call sequence of the package's public entry points, with the
sizes of this repository's own workloads (``scenes.py``), of its tests, or
generic ones:

* ``train``      views of a training step: render, L1 + HEALPix-SSIM loss and
                 backward to every parameter (``render``, ``hssim_loss``)
* ``densify``    one view of a step with depth supervision and density-control
                 statistics, through the lower-level calls of ``Rasterizer``
* ``view``       one rendered view, forward only (``render`` without gradients),
                 with the exact tile lists or the paper's own tile queries
* ``serve``      a backlog of mixed requests through ``Server.serve``
* ``preprocess`` projection of a scene alone
* ``loss``       the loss and its gradient alone, both kinds of window
* ``resample``   a camera image onto the sphere and the sphere back to a camera
                 image

``prepare`` makes the inputs on the GPU from the seed; ``run`` is one pass;
``work`` the bytes and operations a pass cannot do without; ``exact`` the same
outputs in 64 bits from plain torch, where that is affordable.
"""
from __future__ import annotations

import math

import numpy as np
import torch

FULL, FISHEYE, PINHOLE = 0, 1, 2


# ---------------------------------------------------------------------------
# cases
# ---------------------------------------------------------------------------
def listed():
    return [
        # the smallest step a test or a first try makes: bound by launches
        dict(name="train_tiny", op="train", P=2000, sh=0, law="volume", cam=FULL, fov=360.0, order=6, views=1),
        # a small capture seen by a 180-degree fisheye, one view per step
        dict(name="train_fisheye", op="train", P=100_000, sh=3, law="volume", cam=FISHEYE, fov=180.0, order=8, views=1),
        # the benchmark's step: a million Gaussians, four full-sphere views
        dict(name="train_sphere", op="train", P=1_000_000, sh=3, law="log", cam=FULL, fov=360.0, order=9, views=4),
        # a step inside the densification interval of a perspective capture, ragged size
        dict(name="densify_pinhole", op="densify", P=250_007, sh=2, law="log", cam=PINHOLE, fov=75.0, order=10),
        # a high-resolution perspective view of a large scene
        dict(name="view_pinhole", op="view", P=3_000_000, sh=3, law="log", cam=PINHOLE, fov=60.0, order=11, query="", f=0),
        # a panorama through the paper's default tile query
        dict(name="view_ring4", op="view", P=1_000_000, sh=3, law="log", cam=FULL, fov=360.0, order=9, query="ring", f=4),
        # a backlog of requests of every camera model and resolution on a resident scene
        dict(name="serve_mixed", op="serve", P=2_000_000, sh=3, law="log", requests=12, lo=7, hi=10),
        # a panorama with the exact tile lists, without gradients
        dict(name="view_sphere", op="view", P=1_000_000, sh=3, law="log", cam=FULL, fov=360.0, order=9, query="", f=0),
        # the projection of a scene, a stage that a program also calls by itself
        dict(name="preprocess", op="preprocess", P=1_000_000, sh=3, law="log"),
        # the training loss on panoramas, and with the zone-specific windows on a wide fisheye
        dict(name="loss_sphere", op="loss", cam=FULL, fov=360.0, order=9, zones=False),
        dict(name="loss_zones", op="loss", cam=FISHEYE, fov=200.0, order=9, zones=True),
        # ground truth from a panorama, and a rendered sphere back to a panorama
        dict(name="resample_pano", op="resample", cam=FULL, fov=360.0, order=9, W=3040, H=1520),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_cam(rng):
    cam = rng.choice((FULL, FISHEYE, PINHOLE))
    fov = {FULL: 360.0, FISHEYE: rng.uniform(150.0, 220.0), PINHOLE: rng.uniform(50.0, 95.0)}[cam]
    return cam, round(fov, 2)


def draw(rng):
    """A case of the ranges that the listed ones stand for."""
    op = rng.choice(("train", "train", "densify", "view", "view", "serve", "preprocess", "loss", "loss", "resample"))
    cam, fov = _draw_cam(rng)
    sh = rng.randint(0, 3)
    law = rng.choice(("volume", "log"))
    if op == "train":
        return dict(op=op, P=_log_int(rng, 1000, 1_000_000), sh=sh, law=law, cam=cam, fov=fov, order=rng.randint(5, 9),
                    views=rng.randint(1, 4))
    if op == "densify":
        return dict(op=op, P=_log_int(rng, 1000, 1_000_000), sh=sh, law=law, cam=cam, fov=fov,
                    order=rng.randint(6, 10 if cam == PINHOLE else 9))
    if op == "view":
        query = rng.choice(("", "", "ring", "nested"))
        return dict(op=op, P=_log_int(rng, 2000, 3_000_000), sh=sh, law=law, cam=cam, fov=fov,
                    order=rng.randint(6, 11 if cam == PINHOLE else 9), query=query,
                    f=rng.choice((1, 2, 4)) if query else 0)
    if op == "serve":
        return dict(op=op, P=_log_int(rng, 100_000, 2_000_000), sh=sh, law=law, requests=rng.randint(1, 12), lo=7,
                    hi=rng.randint(8, 10))
    if op == "preprocess":
        return dict(op=op, P=_log_int(rng, 1000, 3_000_000), sh=sh, law=law)
    if op == "loss":
        return dict(op=op, cam=cam, fov=fov, order=rng.randint(5, 10), zones=rng.random() < 0.35)
    W = _log_int(rng, 320, 3840)
    return dict(op=op, cam=cam, fov=fov, order=rng.randint(6, 10), W=W, H=max(160, W // 2 + rng.randint(-9, 9)))


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _gen(seed, stream):
    return torch.Generator(device="cuda").manual_seed(1_000_003 * int(seed) + stream)


def _scene(case, seed):
    """Gaussians of scenes.py's laws: [mean, scale, rot, opacity, sh]."""
    P, K = case["P"], (case["sh"] + 1) ** 2
    g = _gen(seed, 1)
    n = lambda *s: torch.randn(*s, generator=g, device="cuda")
    d = n(3, P)
    d = d / d.norm(dim=0, keepdim=True)
    u = torch.rand(P, generator=g, device="cuda")
    r = torch.exp(u * math.log(20.0)) if case["law"] == "log" else (8.0 + 208.0 * u) ** (1.0 / 3.0)
    scale = torch.exp(-3.0 + 0.5 * n(3, P))
    rot = n(4, P)
    rot = rot / rot.norm(dim=0, keepdim=True)
    opacity = torch.sigmoid(n(P))
    sh = 0.2 * n(K, 3, P)
    return [t.contiguous() for t in (d * r, scale, rot, opacity, sh)]


def _fov_y(cam, fov):
    """Radians (x, y): pinholes are 16:9 with square pixels."""
    fx = math.radians(fov)
    if cam == PINHOLE:
        return fx, 2.0 * math.atan(math.tan(fx / 2.0) * 9.0 / 16.0)
    return (2.0 * math.pi, math.pi) if cam == FULL else (fx, fx)


def _camera(rng, cam, fov, order, law):
    """Random pose (centre in a ball of radius 0.5 for the log law, else the
    origin) as a dict of scenes.py's layout."""
    q, r = np.linalg.qr(rng.standard_normal((3, 3)))
    q = q * np.sign(np.diag(r))[None, :]
    if np.linalg.det(q) < 0:
        q[:, 0] = -q[:, 0]
    c = rng.standard_normal(3)
    c *= (0.5 * rng.random() ** (1.0 / 3.0) if law == "log" else 0.0) / np.linalg.norm(c)
    fx, fy = _fov_y(cam, fov)
    W = q.astype(np.float32)
    return dict(W=W, b=(-q @ c).astype(np.float32), center=c.astype(np.float32), cam_type=cam, fov_x=fx, fov_y=fy,
                order=order)


def _cameras(case, seed, n):
    rng = np.random.default_rng([seed, 7])
    return [_camera(rng, case["cam"], case["fov"], case["order"], case.get("law", "volume")) for _ in range(n)]


def _request_cameras(case, seed):
    """The same camera models and resolutions for every seed, other poses."""
    mix, rng = np.random.default_rng([case["requests"], 9]), np.random.default_rng([seed, 8])
    cams = []
    for _ in range(case["requests"]):
        kind = int(mix.integers(0, 3))
        order = int(mix.integers(case["lo"], case["hi"] + 1))
        fov = {FULL: 360.0, FISHEYE: mix.uniform(180.0, 220.0), PINHOLE: mix.uniform(60.0, 90.0)}[kind]
        cams.append(_camera(rng, kind, fov, order, case["law"]))
    return cams


def _noise(seed, stream, *shape):
    return torch.rand(*shape, generator=_gen(seed, stream), device="cuda")


def _images(case, seed, n):
    """A smooth picture and a noisy copy of it, [3][n] in [0, 1]: what a
    render and its target look like to the loss."""
    t = torch.arange(n, device="cuda", dtype=torch.float32) / max(n, 1)
    ref = torch.stack([0.5 + 0.35 * torch.sin(61.0 * (k + 1) * t) for k in range(3)])
    ref = (ref + 0.1 * (_noise(seed, 21, 3, n) - 0.5)).clamp(0.0, 1.0)
    img = (ref + 0.2 * (_noise(seed, 22, 3, n) - 0.5)).clamp(0.0, 1.0)
    return img.contiguous(), ref.contiguous()


def prepare(case, seed):
    from paper_2606_29794_amd.raster import Camera, Gaussians, Rasterizer
    op = case["op"]
    R = Rasterizer("cuda")
    s = dict(op=op, R=R, case=case)
    if op == "serve":
        from paper_2606_29794_amd.serve import Request, Server
        s["server"] = Server(Gaussians(*_scene(case, seed)), R, max_batch=8, n_streams=2, hbm_budget_bytes=64 << 30)
        s["requests"] = [Request(k, 0.0, Camera.from_dict(c)) for k, c in enumerate(_request_cameras(case, seed))]
        for r in s["requests"]:
            R.mask(r.camera)
    elif op == "preprocess":
        s["g"] = Gaussians(*_scene(case, seed))
        s["cam"] = Camera.from_dict(_cameras(dict(case, cam=FULL, fov=360.0, order=9), seed, 1)[0])
    else:
        cams = [Camera.from_dict(c) for c in _cameras(case, seed, case.get("views", 1))]
        s["cams"], s["cam"] = cams, cams[0]
        n = R.mask(cams[0]).n_active
        if op == "train":
            s["params"] = [t.requires_grad_(True) for t in _scene(case, seed)]
            s["g"] = Gaussians(*[p.detach() for p in s["params"]])
            s["targets"] = [_noise(seed, 100 + v, 3, n) for v in range(len(cams))]
            R.ssim_tables(cams[0])
        elif op == "densify":
            s["g"] = Gaussians(*_scene(case, seed))
            s["d_rgb"] = (_noise(seed, 31, 3, n) - 0.5) / n
            s["d_inv"] = (_noise(seed, 32, n) - 0.5) / n
        elif op == "view":
            s["g"] = Gaussians(*_scene(case, seed))
        elif op == "loss":
            img, s["ref"] = _images(case, seed, n)
            s["img"] = img.requires_grad_(True)
            R.ssim_tables(s["cam"])
        else:
            s["photo"] = _noise(seed, 41, 3, case["H"], case["W"])
            s["sphere"] = _noise(seed, 42, 3, n)
    torch.cuda.synchronize()
    return s


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------
def _run_train(s):
    from paper_2606_29794_amd.render import hssim_loss, render
    R, params, cams = s["R"], s["params"], s["cams"]
    for p in params:
        p.grad = None
    ahead = R.prefetch(s["g"], cams) if len(cams) > 1 else None
    out = []
    for v, cam in enumerate(cams):
        rgb, _ = render(*params, cam, R, fused_grad=True, prepared=ahead.get(v) if ahead else None)
        loss, stats = hssim_loss(rgb, s["targets"][v], cam, 0.2, R)
        loss.backward()
        out.append(stats)
    R.verify(block=False)
    return out + [p.grad for p in params]


def _run_densify(s):
    from paper_2606_29794_amd.raster import Gaussians
    R, g, cam = s["R"], s["g"], s["cam"]
    st = R.forward(g, cam, want_depth=True)
    dev = g.mean.device
    acc = torch.zeros((10, g.P), dtype=torch.float32, device=dev)
    R.backward_pixels(st, s["d_rgb"], None, acc, s["d_inv"])
    z = torch.zeros_like
    grads = Gaussians(z(g.mean), z(g.scale), z(g.rot), z(g.opacity), z(g.sh))
    R.backward_preprocess(g, cam, acc, grads)
    rs_max, accum = torch.zeros(g.P, device=dev), torch.zeros(g.P, device=dev)
    count = torch.zeros(g.P, dtype=torch.int32, device=dev)
    R.density_stats(st, acc, rs_max, accum, count)
    R.verify(block=False)
    return [st.rgb, st.T, st.inv_depth, grads.mean, grads.scale, grads.rot, grads.opacity, grads.sh, rs_max, accum, count]


def run(s):
    op, R = s["op"], s["R"]
    if op == "train":
        return _run_train(s)
    if op == "densify":
        return _run_densify(s)
    if op == "view":
        from paper_2606_29794_amd.render import render
        g, c = s["g"], s["case"]
        with torch.no_grad():
            rgb, T = render(g.mean, g.scale, g.rot, g.opacity, g.sh, s["cam"], R,
                            query=(c["query"], c["f"]) if c["query"] else None)
        R.verify(block=False)
        return [rgb, T]
    if op == "serve":
        stats = s["server"].serve(s["requests"], realtime=False, keep_outputs=True)
        return [t for r in stats.results for t in (r.rgb, r.T)]
    if op == "preprocess":
        return list(R.projected_arrays(R.preprocess(s["g"], s["cam"]), s["g"].P))
    if op == "loss":
        from paper_2606_29794_amd.render import hssim_loss
        img = s["img"]
        img.grad = None
        loss, stats = hssim_loss(img, s["ref"], s["cam"], 0.2, R, zones=s["case"]["zones"])
        loss.backward()
        return [stats, img.grad]
    on_sphere, ok = R.image_to_sphere(s["photo"], s["cam"], want_valid=True)
    image, ok2 = R.sphere_to_image(s["sphere"], s["cam"], s["case"]["W"], s["case"]["H"], want_valid=True)
    return [on_sphere, ok, image, ok2]


# ---------------------------------------------------------------------------
# work
# ---------------------------------------------------------------------------
def _active(cam, fov, order):
    """Active pixels, from the solid angle of the field of view."""
    npix = 12 * 4 ** order
    fx, fy = _fov_y(cam, fov)
    if cam == FULL:
        return npix
    if cam == FISHEYE:
        return int(npix * 0.5 * (1.0 - math.cos(min(fx / 2.0, math.pi))))
    return int(npix * 4.0 * math.asin(math.sin(fx / 2.0) * math.sin(fy / 2.0)) / (4.0 * math.pi))


def _composited(case):
    """Gaussians composited per pixel: the scene's 3-sigma footprints over a
    pixel, at most the 75 after which a pixel of a dense scene is opaque."""
    inv_r2 = 0.1665 if case["law"] == "log" else 0.0577
    return min(75.0, case["P"] * 9.0 * math.pi * math.exp(-5.75) * inv_r2 / (4.0 * math.pi))


def work(case):
    op = case["op"]
    if op == "serve":
        par = case["P"] * 4 * (11 + 3 * (case["sh"] + 1) ** 2)
        n = [_active(c["cam_type"], math.degrees(c["fov_x"]), c["order"]) for c in _request_cameras(case, 0)]
        return dict(bytes=par + 16 * sum(n), flops=sum(n) * _composited(case) * 54)
    if op == "preprocess":
        return dict(bytes=case["P"] * (4 * (11 + 3 * (case["sh"] + 1) ** 2) + 88), flops=case["P"] * 400)
    n = _active(case["cam"], case["fov"], case["order"])
    if op == "loss":
        return dict(bytes=36 * n, flops=1190 * n if not case["zones"] else 1190 * n + n / 3 * 121 * 60)
    if op == "resample":
        px = case["W"] * case["H"]
        return dict(bytes=12 * (px + n) + 13 * (px + n), flops=200 * (px + n))
    par = case["P"] * 4 * (11 + 3 * (case["sh"] + 1) ** 2)
    pairs = n * _composited(case)
    if op == "view":
        return dict(bytes=par + 16 * n, flops=54 * pairs)
    if op == "densify":
        return dict(bytes=2 * par + 12 * case["P"] + 36 * n, flops=(54 + 114) * pairs)
    v = case["views"]
    return dict(bytes=2 * par + v * 12 * n, flops=v * ((54 + 114) * pairs + 1190 * n))


# ---------------------------------------------------------------------------
# the same outputs in 64 bits
# ---------------------------------------------------------------------------
F8 = torch.float64


def _bits(v, get):
    """Every second bit of v gathered (get) or spread (not get)."""
    out = torch.zeros_like(v)
    for k in range(16):
        out |= ((v >> (2 * k)) & 1) << k if get else ((v >> k) & 1) << (2 * k)
    return out


def _nest_xyf(order, p):
    f = p >> (2 * order)
    q = p & ((1 << (2 * order)) - 1)
    return _bits(q, True), _bits(q >> 1, True), f


def _xyf_nest(order, x, y, f):
    return (f << (2 * order)) + (_bits(x, False) | (_bits(y, False) << 1))


def _ring(order, p):
    """Ring (1 .. 4N-1) and 0-based position along it of nested pixels."""
    x, y, f = _nest_xyf(order, p)
    N = 1 << order
    row, col = f >> 2, f & 3
    ring = (row + 2) * N - x - y - 1
    lon = torch.where(row == 1, 2 * col, 2 * col + 1)
    cap = (ring < N) | (ring > 3 * N)
    nr = torch.where(ring < N, ring, torch.where(ring > 3 * N, 4 * N - ring, torch.full_like(ring, N)))
    shift = torch.where(cap, torch.zeros_like(ring), (ring - N) & 1)
    j = (lon * nr + x - y + 1 + shift) // 2 - 1
    return ring, j % (4 * nr)


def _ring_geometry(order, ring):
    """(z, sin theta, pixels, offset of pixel 0 in pixels) of rings."""
    N = 1 << order
    cap = (ring < N) | (ring > 3 * N)
    nr = torch.where(ring < N, ring, torch.where(ring > 3 * N, 4 * N - ring, torch.full_like(ring, N)))
    h = nr.to(F8) ** 2 / (3.0 * N * N)
    z = torch.where(cap, torch.where(ring < N, 1.0 - h, h - 1.0), (2 * N - ring).to(F8) * 2.0 / (3.0 * N))
    st = torch.where(cap, torch.sqrt(h * (2.0 - h)), torch.sqrt((1.0 - z) * (1.0 + z)))
    off = torch.where(cap | (((ring - N) & 1) == 0), 0.5, 0.0).to(F8)
    return z, st, 4 * nr, off


def _directions(order, p):
    """Unit pixel-centre directions [3][n], pole on +y, longitude atan2(x, z)."""
    ring, pos = _ring(order, p)
    z, st, n, off = _ring_geometry(order, ring)
    phi = (pos.to(F8) + off) * (2.0 * math.pi) / n.to(F8)
    return torch.stack([st * torch.sin(phi), z, st * torch.cos(phi)])


def _active_pixels(cam, order):
    p = torch.arange(12 * 4 ** order, device="cuda")
    if cam["cam_type"] == FULL:
        return p
    d = _directions(order, p)
    fx, fy = float(np.float32(cam["fov_x"])), float(np.float32(cam["fov_y"]))
    if cam["cam_type"] == PINHOLE:
        ok = (d[2] > 0) & (d[0].abs() <= math.tan(fx / 2) * d[2]) & (d[1].abs() <= math.tan(fy / 2) * d[2])
    else:
        gam = torch.atan2(d[1], d[0])
        weff = torch.sqrt((fx / math.pi * torch.cos(gam)) ** 2 + (fy / math.pi * torch.sin(gam)) ** 2)
        ok = torch.acos(d[2].clamp(-1, 1)) <= 0.5 * math.pi * weff
    return p[ok]


def _sh_basis(deg, d):
    x, y, z = d
    Y = [torch.full_like(x, 0.5 / math.sqrt(math.pi))]
    if deg > 0:
        k = math.sqrt(3.0 / (4.0 * math.pi))
        Y += [k * y, k * z, k * x]
    if deg > 1:
        k = 0.5 * math.sqrt(15.0 / math.pi)
        Y += [k * x * y, k * y * z, 0.25 * math.sqrt(5.0 / math.pi) * (3 * z * z - 1), k * x * z, 0.5 * k * (x * x - y * y)]
    if deg > 2:
        a, b = 0.25 * math.sqrt(35.0 / (2.0 * math.pi)), 0.5 * math.sqrt(105.0 / math.pi)
        c, e = 0.25 * math.sqrt(21.0 / (2.0 * math.pi)), 0.25 * math.sqrt(7.0 / math.pi)
        Y += [a * y * (3 * x * x - y * y), b * x * y * z, c * y * (5 * z * z - 1), e * z * (5 * z * z - 3),
              c * x * (5 * z * z - 1), 0.5 * b * z * (x * x - y * y), a * x * (x * x - 3 * y * y)]
    return torch.stack(Y)


def _frame(om, ph):
    so, co, sp, cp = torch.sin(om), torch.cos(om), torch.sin(ph), torch.cos(ph)
    o = torch.zeros_like(so)
    return torch.stack([cp * so, sp, cp * co]), torch.stack([co, o, -so]), torch.stack([-sp * so, cp, -sp * co])


def _project(params, deg, cam):
    """Stage 1 in 64 bits, differentiable: the frame (om, ph) that the offsets
    use is kept apart from the one in the covariance."""
    mean, scale, rot, opacity, sh = params
    W = torch.as_tensor(np.asarray(cam["W"], np.float64), device="cuda")
    b = torch.as_tensor(np.asarray(cam["b"], np.float64), device="cuda")[:, None]
    c = torch.as_tensor(np.asarray(cam["center"], np.float64), device="cuda")[:, None]
    t = W @ mean + b
    r = t.norm(dim=0)
    om, ph = torch.atan2(t[0], t[2]), torch.atan2(t[1], torch.sqrt(t[0] ** 2 + t[2] ** 2))
    _, eo, ep = _frame(om, ph)
    w, x, y, z = rot / rot.norm(dim=0, keepdim=True)
    Rm = [[1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y)],
          [2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x)],
          [2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)]]
    V = []
    for e in (eo, ep):
        eW = W.T @ e
        V.append(torch.stack([(eW[0] * Rm[0][k] + eW[1] * Rm[1][k] + eW[2] * Rm[2][k]) * scale[k] / r for k in range(3)]))
    sa, sb, sc = (V[0] * V[0]).sum(0), (V[0] * V[1]).sum(0), (V[1] * V[1]).sum(0)
    cr = torch.linalg.cross(V[0].T, V[1].T)
    det = (cr * cr).sum(1)
    lmax = 0.5 * (sa + sc) + torch.sqrt((0.5 * (sa - sc)) ** 2 + sb * sb)
    radius = torch.clamp(3.0 * torch.sqrt(lmax), max=math.pi)
    v = mean - c
    Y = _sh_basis(deg, v / v.norm(dim=0, keepdim=True))
    rgb = torch.clamp(0.5 + (sh * Y[:, None]).sum(0), min=0.0)
    return dict(om=om, ph=ph, r=r, conic=torch.stack([sc / det, -sb / det, sa / det]), radius=radius, rgb=rgb,
                opacity=opacity)


def _composite(pr, om, ph, dirs):
    """rgb [3][n], T [n] and inverse depth [n] at directions dirs, brute force
    over Gaussians in front-to-back order."""
    u, eo, ep = _frame(om, ph)
    a, b, c = dirs.T @ eo, dirs.T @ ep, dirs.T @ u
    s = torch.sqrt(a * a + b * b).clamp_min(1e-300)
    k = torch.atan2(s, c) / s
    A, B, C = pr["conic"]
    q = (A * a * a + 2 * B * a * b + C * b * b) * k * k
    alpha = torch.where(q <= 9.0, torch.clamp(pr["opacity"] * torch.exp(-0.5 * q), max=float(np.float32(0.99))),
                        torch.zeros_like(q))
    lt = torch.cumsum(torch.log1p(-alpha), 1)
    before = torch.exp(torch.cat([torch.zeros_like(lt[:, :1]), lt[:, :-1]], 1))
    live = before.detach() >= float(np.float32(1e-4))
    w = torch.where(live, before * alpha, torch.zeros_like(alpha))
    T = torch.exp(torch.where(live, torch.log1p(-alpha), torch.zeros_like(alpha)).sum(1))
    return pr["rgb"] @ w.T, T, w @ (1.0 / pr["r"])


def _chunks(n, P):
    step = max(64, 6_000_000 // P)
    return [slice(i, min(n, i + step)) for i in range(0, n, step)]


def _exact_render(case, seed, cam, upstream):
    """(rgb, T, inverse depth, radius, direction gradients, parameter
    gradients) of one view; upstream(rgb, T) gives (dL/drgb, dL/dinv) or None."""
    params = [t.to(F8).requires_grad_(True) for t in _scene(case, seed)]
    pr = _project(params, case["sh"], cam)
    keys = ("om", "ph", "r", "conic", "rgb", "opacity")
    leaf = {k: pr[k].detach().requires_grad_(True) for k in keys}
    order = torch.argsort(leaf["r"].detach().float(), stable=True)
    srt = {k: v[..., order] for k, v in leaf.items()}
    dirs = _directions(cam["order"], _active_pixels(cam, cam["order"]))
    n = dirs.shape[1]
    with torch.no_grad():
        out = [_composite(srt, srt["om"], srt["ph"], dirs[:, c]) for c in _chunks(n, case["P"])]
    rgb, T, inv = (torch.cat([o[k] for o in out], -1) for k in range(3))
    up = upstream(rgb, T)
    if up is None:
        return rgb, T, inv, None, None, None
    for c in _chunks(n, case["P"]):
        srt = {k: v[..., order] for k, v in leaf.items()}
        o = _composite(srt, srt["om"], srt["ph"], dirs[:, c])
        L = (o[0] * up[0][:, c]).sum()
        if up[1] is not None:
            L = L + (o[2] * up[1][c]).sum()
        L.backward()
    torch.autograd.backward([pr[k] for k in keys if leaf[k].grad is not None],
                            [leaf[k].grad for k in keys if leaf[k].grad is not None])
    return rgb, T, inv, pr["radius"].detach(), (leaf["om"].grad, leaf["ph"].grad, pr["ph"].detach()), [p.grad for p in params]


# neighbouring face beyond the edges (sx, sy) of a face: row of faces, column
# step, and the coordinates there, for faces of the northern, equatorial and
# southern row; the corners that are not listed have no pixel
_BEYOND = (
    {(1, 0): (0, 1, lambda x, y, N: (y, 2 * N - 1 - x)), (-1, 0): (1, 0, lambda x, y, N: (x + N, y)),
     (0, 1): (0, 3, lambda x, y, N: (2 * N - 1 - y, x)), (0, -1): (1, 1, lambda x, y, N: (x, y + N)),
     (1, 1): (0, 2, lambda x, y, N: (2 * N - 1 - x, 2 * N - 1 - y)), (-1, -1): (2, 0, lambda x, y, N: (x + N, y + N))},
    {(1, 0): (0, 0, lambda x, y, N: (x - N, y)), (-1, 0): (2, 3, lambda x, y, N: (x + N, y)),
     (0, 1): (0, 3, lambda x, y, N: (x, y - N)), (0, -1): (2, 0, lambda x, y, N: (x, y + N)),
     (1, -1): (1, 1, lambda x, y, N: (x - N, y + N)), (-1, 1): (1, 3, lambda x, y, N: (x + N, y - N))},
    {(1, 0): (1, 1, lambda x, y, N: (x - N, y)), (-1, 0): (2, 3, lambda x, y, N: (y, -1 - x)),
     (0, 1): (1, 0, lambda x, y, N: (x, y - N)), (0, -1): (2, 1, lambda x, y, N: (-1 - y, x)),
     (1, 1): (0, 0, lambda x, y, N: (x - N, y - N)), (-1, -1): (2, 2, lambda x, y, N: (-1 - x, -1 - y))},
)


def _chart(order, f, x, y):
    """Nested pixels at face-extended coordinates, -1 where there is none."""
    N = 1 << order
    sx, sy = (x >= N).long() - (x < 0).long(), (y >= N).long() - (y < 0).long()
    out = torch.where((sx == 0) & (sy == 0), _xyf_nest(order, x.clamp(0, N - 1), y.clamp(0, N - 1), f),
                      torch.full_like(x, -1))
    for row in range(3):
        for (ex, ey), (to, dc, go) in _BEYOND[row].items():
            m = ((f >> 2) == row) & (sx == ex) & (sy == ey)
            if bool(m.any()):
                X, Y = go(x[m], y[m], N)
                out[m] = _xyf_nest(order, X, Y, 4 * to + (((f[m] & 3) + dc) & 3))
    return out


def _exact_loss(img, ref, cam, zones, lam=0.2):
    """(stats [3], dL/dimg [3][n]) of the loss in 64 bits."""
    order = cam["order"]
    act = _active_pixels(cam, order)
    n = act.numel()
    slot = torch.full((12 * 4 ** order,), -1, dtype=torch.long, device="cuda")
    slot[act] = torch.arange(n, device="cuda")
    x, y, f = _nest_xyf(order, act)
    N = 1 << order
    ring, _ = _ring(order, act)
    polar = ((ring < N) | (ring > 3 * N)) if zones else None
    dirs = _directions(order, act) if zones else None
    wscale = 1.0 / (2.0 * 1.5 ** 2 * 4.0 * math.pi / (12.0 * 4 ** order))
    img, ref = img.to(F8), ref.to(F8)

    def taps():
        for dy in range(-5, 6):
            for dx in range(-5, 6):
                q = _chart(order, f, x + dx, y + dy)
                k = torch.where(q >= 0, slot[q.clamp_min(0)], q)
                w = torch.full((n,), math.exp(-(dx * dx + dy * dy) / 4.5), dtype=F8, device="cuda")
                kk = k.clamp_min(0)
                if zones:
                    h = 0.5 * (dirs - dirs[:, kk]).norm(dim=0)
                    d = 2.0 * torch.asin(h.clamp(max=1.0))
                    w = torch.where(polar, torch.exp(-d * d * wscale), w)
                yield torch.where(k >= 0, w, torch.zeros_like(w)), kk

    Z, S = torch.zeros(n, dtype=F8, device="cuda"), [torch.zeros_like(img) for _ in range(5)]
    for w, k in taps():
        a, b = img[:, k], ref[:, k]
        Z += w
        for s, v in zip(S, (a, b, a * a, b * b, a * b)):
            s += w * v
    m = [(s / Z).requires_grad_(True) for s in S]
    mx, my, xx, yy, xy = m
    C1, C2 = float(np.float32(1e-4)), float(np.float32(9e-4))
    ssim = ((2 * mx * my + C1) * (2 * (xy - mx * my) + C2)) / ((mx * mx + my * my + C1) * (xx - mx * mx + yy - my * my + C2))
    g = torch.autograd.grad(ssim.sum(), [mx, xx, xy])
    g = [t / Z for t in g]
    dimg = torch.zeros_like(img)
    for w, k in taps():
        dimg.index_add_(1, k, w * (g[0] + 2 * img[:, k] * g[1] + ref[:, k] * g[2]))
    l1, mean = (img - ref).abs().mean(), ssim.detach().mean()
    d = ((1 - lam) * torch.sign(img - ref) - lam * dimg) / (3.0 * n)
    return torch.stack([mean, l1, (1 - lam) * l1 + lam * (1 - mean)]), d


def _exact_preprocess(case, seed):
    cam = _cameras(dict(case, cam=FULL, fov=360.0, order=9), seed, 1)[0]
    with torch.no_grad():
        pr = _project([t.to(F8) for t in _scene(case, seed)], case["sh"], cam)
        u, eo, ep = _frame(pr["om"], pr["ph"])
        half = torch.sin(0.5 * torch.clamp(pr["radius"] + float(np.float32(1e-6)), max=math.pi))
        rec = torch.stack([u[0], u[1], u[2], pr["opacity"], eo[0], eo[2], ep[0], ep[1], ep[2], *pr["conic"], *pr["rgb"], half])
    return [rec.T.contiguous(), pr["r"], pr["radius"]]


def _exact_resample(case, seed):
    cam = _cameras(case, seed, 1)[0]
    order, W, H, kind = case["order"], case["W"], case["H"], case["cam"]
    act = _active_pixels(cam, order)
    photo, sphere = _noise(seed, 41, 3, H, W).to(F8), _noise(seed, 42, 3, act.numel()).to(F8)
    fx, fy = float(np.float32(cam["fov_x"])), float(np.float32(cam["fov_y"]))
    lx, ly = (W / (2 * math.tan(fx / 2)), H / (2 * math.tan(fy / 2))) if kind == PINHOLE else (W / math.pi, H / math.pi)
    # photo -> sphere: every active pixel centre projected into the image
    d = _directions(order, act)
    if kind == FULL:
        u = (torch.atan2(d[0], d[2]) + math.pi) * W / (2 * math.pi)
        v = (0.5 * math.pi - torch.asin(d[1].clamp(-1, 1))) * H / math.pi
        ok = torch.ones_like(u, dtype=torch.bool)
    elif kind == PINHOLE:
        u, v = 0.5 * W + lx * d[0] / d[2], 0.5 * H - ly * d[1] / d[2]
        ok = (d[2] > 0) & (u >= 0) & (u <= W) & (v >= 0) & (v <= H)
    else:
        gam = torch.atan2(d[1], d[0])
        rm = torch.acos(d[2].clamp(-1, 1)) / torch.sqrt((fx / math.pi * torch.cos(gam)) ** 2 + (fy / math.pi * torch.sin(gam)) ** 2)
        u, v = 0.5 * W + lx * rm * torch.cos(gam), 0.5 * H - ly * rm * torch.sin(gam)
        ok = rm <= 0.5 * math.pi
    x0, y0 = torch.floor(u - 0.5), torch.floor(v - 0.5)
    ax, ay = u - 0.5 - x0, v - 0.5 - y0
    col = lambda t: (t.long() % W) if kind == FULL else t.long().clamp(0, W - 1)
    row = lambda t: t.long().clamp(0, H - 1)
    at = lambda yy, xx: photo[:, row(yy), col(xx)]
    on = (1 - ay) * ((1 - ax) * at(y0, x0) + ax * at(y0, x0 + 1)) + ay * ((1 - ax) * at(y0 + 1, x0) + ax * at(y0 + 1, x0 + 1))
    on = torch.where(ok, on, torch.zeros_like(on))
    # sphere -> image: bilinear between the two enclosing rings
    npix, N = 12 * 4 ** order, 1 << order
    slot = torch.full((npix,), -1, dtype=torch.long, device="cuda")
    slot[act] = torch.arange(act.numel(), device="cuda")
    rings = torch.arange(4 * N + 1, device="cuda")
    z, st, cnt, off = _ring_geometry(order, rings[1:4 * N])
    theta_r = torch.cat([torch.zeros(1, dtype=F8, device="cuda"), torch.atan2(st, z), torch.full((1,), math.pi, dtype=F8, device="cuda")])
    cnt, off = (torch.cat([t[:1], t, t[-1:]]) for t in (cnt, off))
    cnt[0] = cnt[-1] = 0
    first = torch.cumsum(cnt, 0) - cnt
    p = torch.arange(npix, device="cuda")
    ring, pos = _ring(order, p)
    by_ring = torch.empty_like(slot)
    by_ring[first[ring] + pos] = slot
    jj, ii = torch.meshgrid(torch.arange(H, device="cuda", dtype=F8), torch.arange(W, device="cuda", dtype=F8), indexing="ij")
    uu, vv = ii.reshape(-1) + 0.5, jj.reshape(-1) + 0.5
    inside = torch.ones_like(uu, dtype=torch.bool)
    if kind == FULL:
        om, ph = 2 * math.pi * uu / W - math.pi, 0.5 * math.pi - math.pi * vv / H
        d, _, _ = _frame(om, ph)
    else:
        mx, my = (uu - 0.5 * W) / lx, -(vv - 0.5 * H) / ly
        if kind == PINHOLE:
            d = torch.stack([mx, my, torch.ones_like(mx)])
            d = d / d.norm(dim=0)
        else:
            rm, gam = torch.sqrt(mx * mx + my * my), torch.atan2(my, mx)
            psi = rm * torch.sqrt((fx / math.pi * torch.cos(gam)) ** 2 + (fy / math.pi * torch.sin(gam)) ** 2)
            d = torch.stack([torch.sin(psi) * torch.cos(gam), torch.sin(psi) * torch.sin(gam), torch.cos(psi)])
            inside = rm <= 0.5 * math.pi
    theta, phi = torch.atan2(torch.sqrt(d[0] ** 2 + d[2] ** 2), d[1]), torch.atan2(d[0], d[2]) % (2 * math.pi)
    i1 = (torch.searchsorted(theta_r, theta, right=True) - 1).clamp(0, 4 * N - 1)
    wt = (theta - theta_r[i1]) / (theta_r[i1 + 1] - theta_r[i1])
    total, ws = torch.zeros(3, uu.numel(), dtype=F8, device="cuda"), torch.zeros_like(uu)

    def add(i, j, w):
        nonlocal total, ws
        k = by_ring[first[i] + j]
        w = torch.where((k >= 0) & inside, w, torch.zeros_like(w))
        total += w * sphere[:, k.clamp_min(0)]
        ws += w

    for i, wr in ((i1, 1 - wt), (i1 + 1, wt)):
        pole, near = (i == 0) | (i == 4 * N), i.clamp(1, 4 * N - 1)
        c = cnt[near]
        t = phi * c.to(F8) / (2 * math.pi) - off[near]
        j = torch.floor(t)
        fr, j = t - j, j.long()
        add(near, j % c, torch.where(pole, torch.zeros_like(wr), wr * (1 - fr)))
        add(near, (j + 1) % c, torch.where(pole, torch.zeros_like(wr), wr * fr))
        for k in range(4):  # the pole: the mean of its ring's four pixels
            add(near, torch.full_like(j, k) % c, torch.where(pole, 0.25 * wr, torch.zeros_like(wr)))
    image = torch.where(ws > 0, total / ws.clamp_min(1e-300), torch.zeros_like(total))
    return [on, None, image.view(3, H, W), None]


def exact(case, seed):
    op = case["op"]
    if op == "preprocess":
        return _exact_preprocess(case, seed)
    if op == "resample":
        return _exact_resample(case, seed)
    if op == "serve" or (op == "view" and case["query"]):
        return None
    cams = _cameras(case, seed, case.get("views", 1))
    n = _active(case["cam"], case["fov"], case["order"])
    if op == "loss":
        img, ref = _images(case, seed, _active_pixels(cams[0], case["order"]).numel())
        return list(_exact_loss(img, ref, cams[0], case["zones"]))
    if case["P"] * n * len(cams) > 400_000_000:  # brute force over every pair
        return None
    n = _active_pixels(cams[0], case["order"]).numel()
    if op == "view":
        rgb, T, _, _, _, _ = _exact_render(case, seed, cams[0], lambda *a: None)
        return [rgb, T]
    if op == "train":
        stats, grads = [], None
        for v, cam in enumerate(cams):
            target, keep = _noise(seed, 100 + v, 3, n), []

            def upstream(rgb, T):
                st, d = _exact_loss(rgb, target, cam, False)
                keep.append(st)
                return d, None

            gr = _exact_render(case, seed, cam, upstream)[5]
            stats.append(keep[0])
            grads = gr if grads is None else [a + b for a, b in zip(grads, gr)]
        return stats + grads
    up = ((_noise(seed, 31, 3, n) - 0.5) / n).to(F8), ((_noise(seed, 32, n) - 0.5) / n).to(F8)
    rgb, T, inv, radius, (g_om, g_ph, ph), grads = _exact_render(case, seed, cams[0], lambda *a: up)
    # the statistics of Gaussians that reach no tile stay at zero: which ones
    # do is a matter of the tile lists, not of 64-bit arithmetic
    return [rgb, T, inv, *grads, None, torch.sqrt((g_om / torch.cos(ph)) ** 2 + g_ph ** 2), None]

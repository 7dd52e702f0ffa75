"""The work that users have this renderer do, as measurable cases.

A case is a dict of plain values.  `kind` picks the entry point:

    frame   Renderer.render of an explicit scene: per-cell (duplex), the
            per-Gaussian comparison path (alpha) or LC-WSR weights, fixed
            members per cell or CSR offsets
    neural  Renderer.render_neural: decode of the visible cells, then a frame
    train   DuplexRenderPlanar + L1SsimLoss + backward: a differentiation step
    loss    Renderer.loss_l1_ssim alone
    sort    Renderer.sort_pairs on caller data
    serve   a burst of requests through the serving runtime

Scenes follow the distributions of scenes.py (tiny, clustered, aerial-scale,
ragged, neural), drawn on the GPU from the seed so that making them is quick.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2508_03180_amd import _capi as capi
from paper_2508_03180_amd import scenes
from paper_2508_03180_amd.renderer import (DeviceScene, DuplexRenderPlanar, L1SsimLoss, NeuralDeviceScene, Renderer)
from paper_2508_03180_amd.serving import Server

DEV = "cuda:0"
LAMBDA = 0.2   # weight of the SSIM term of the training loss
TAU = 8.0      # LC-WSR depth scale of the clustered scene


def listed():
    return [
        # a thumbnail of a small scene, called one at a time with the default
        # checks: launches and latency
        dict(name="frame_tiny", kind="frame", scene="tiny", cells=2000, K=8, degree=0, width=256, height=256,
             view=3, mode="duplex", check=True),
        # a pruned scene (members per cell differ) in a preview window of odd size
        dict(name="frame_ragged_720p", kind="frame", scene="ragged", cells=20000, K=12, degree=2, width=1283,
             height=717, view=7, mode="duplex", check=False),
        # the benchmark's orbit frame: 1M Gaussians at full HD
        dict(name="frame_1080p", kind="frame", scene="mid", cells=100000, K=10, degree=3, width=1920, height=1080,
             view=10, mode="duplex", check=False),
        # the per-Gaussian comparison path on the same scene
        dict(name="frame_alpha_1080p", kind="frame", scene="mid", cells=100000, K=10, degree=3, width=1920,
             height=1080, view=10, mode="alpha", check=False),
        # a street-level 4K view of a 6M-Gaussian aerial-scale scene
        dict(name="frame_large_4k", kind="frame", scene="large", cells=600000, K=10, degree=3, width=3840,
             height=2160, view=3, mode="duplex", check=False),
        # an orbit frame whose Gaussians are decoded from cell features
        dict(name="neural_1080p", kind="neural", cells=100000, K=10, F=32, H=32, width=1920, height=1080, view=10),
        # a wider decoder on a smaller scene and window
        dict(name="neural_wide_480p", kind="neural", cells=20000, K=4, F=48, H=64, width=641, height=479, view=4),
        # one view of a training step at full HD
        dict(name="train_1080p", kind="train", scene="mid", cells=100000, K=10, degree=3, width=1920, height=1080,
             view=0),
        # a training step on a small scene and image
        dict(name="train_small", kind="train", scene="tiny", cells=2000, K=8, degree=3, width=301, height=203,
             view=2),
        # the training loss and its gradient alone, on an image of odd size
        dict(name="loss_1600", kind="loss", channels=3, width=1599, height=1201, grad=True),
        # the onesweep sort of a caller's pairs
        dict(name="sort_4m", kind="sort", n=4000037, bits=47),
        # a burst of mixed requests through the server (graph replay, four slots)
        dict(name="serve_burst", kind="serve", cells=20000, K=10, requests=12),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["frame", "frame", "frame", "frame", "neural", "train", "loss", "sort"])
    w, h = _log_int(rng, 64, 1920), _log_int(rng, 48, 1080)
    view = rng.randrange(60)
    if kind == "frame":
        scene = rng.choice(["tiny", "mid", "mid", "ragged", "large"])
        K = _log_int(rng, 2, 32)
        cells = _log_int(rng, 500, {"tiny": 20000, "ragged": 40000}.get(scene, 1000000 // K))
        return dict(kind="frame", scene=scene, cells=cells, K=K, degree=rng.randrange(4), width=w, height=h,
                    view=view, mode=rng.choice(["duplex", "duplex", "duplex", "alpha", "lcwsr"]),
                    check=rng.random() < 0.5)
    if kind == "neural":
        F, H = rng.choice([(32, 32), (rng.randrange(8, 65), rng.randrange(8, 65))])
        K = _log_int(rng, 2, 16)
        return dict(kind="neural", cells=_log_int(rng, 1000, 1000000 // K), K=K, F=F, H=H, width=w, height=h,
                    view=view)
    if kind == "train":
        K = _log_int(rng, 2, 32)
        scene = rng.choice(["tiny", "mid"])
        return dict(kind="train", scene=scene, cells=_log_int(rng, 500, 20000 if scene == "tiny" else 1000000 // K),
                    K=K, degree=rng.randrange(4), width=w, height=h, view=view)
    if kind == "loss":
        return dict(kind="loss", channels=rng.choice([1, 3, 3]), width=w, height=h, grad=rng.random() < 0.7)
    return dict(kind="sort", n=_log_int(rng, 1000, 4000000), bits=rng.randrange(8, 65))


# ------------------------------------------------------------------ inputs

class _Rng:
    def __init__(self, seed):
        self.g = torch.Generator(device=DEV).manual_seed(int(seed))

    def normal(self, *shape, mean=0.0, std=1.0):
        return torch.randn(shape, device=DEV, generator=self.g) * std + mean

    def uniform(self, *shape, lo=0.0, hi=1.0):
        return torch.rand(shape, device=DEV, generator=self.g) * (hi - lo) + lo

    def integers(self, lo, hi, *shape):
        return torch.randint(lo, hi, shape, device=DEV, generator=self.g)


def _unit(x):
    return x / x.norm(dim=0, keepdim=True)


def _ball(r, n):
    return _unit(r.normal(3, n)) * r.uniform(n) ** (1.0 / 3.0)


def _rotmat(q):
    """[3][3] rows of the rotation of quaternions q [4, n] (w, x, y, z)."""
    w, x, y, z = q / torch.sqrt((q * q).sum(0))
    return [[1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y)],
            [2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x)],
            [2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)]]


def _rotate(q, v):
    R = _rotmat(q)
    return torch.stack([R[i][0] * v[0] + R[i][1] * v[1] + R[i][2] * v[2] for i in range(3)])


def _clustered(r, N):
    """50 anisotropic clusters and a tenth of uniform background."""
    n_cl = 50
    wts = torch.cumsum(-torch.log(r.uniform(n_cl, lo=1e-6)), 0)
    which = torch.searchsorted(wts / wts[-1], r.uniform(N, hi=0.999999))
    mean, rot = r.uniform(3, n_cl, lo=-1.0, hi=1.0), _unit(r.normal(4, n_cl))
    std = torch.exp(r.uniform(3, n_cl, lo=math.log(0.03), hi=math.log(0.3)))
    pos = mean[:, which] + _rotate(rot[:, which], r.normal(3, N) * std[:, which])
    bg = r.uniform(N) < 0.1
    return torch.where(bg, r.uniform(3, N, lo=-1.5, hi=1.5), pos)


def _cells(r, kind, N):
    """cell_pos, cell_scale, cell_rot, cell_v_sh, per-cell radius (large)."""
    radius = None
    if kind == "large":
        y = -3.0 * torch.log(1.0 - r.uniform(N) * (1.0 - math.exp(-20.0 / 3.0)))
        xz = r.uniform(2, N, lo=-100.0, hi=100.0)
        pos = torch.stack([xz[0], y, xz[1]])
        radius = torch.exp(r.uniform(N, lo=math.log(0.005), hi=math.log(5.0)))
        scale = radius * torch.exp(r.normal(3, N, std=0.3))
    elif kind in ("mid", "neural"):
        pos, scale = _clustered(r, N), torch.exp(r.normal(3, N, mean=-4.0, std=0.3))
    else:
        pos, scale = r.uniform(3, N, lo=-1.0, hi=1.0), torch.exp(r.normal(3, N, mean=-3.0, std=0.3))
    vsh = r.normal(4, N, std=0.3)
    vsh[0] = r.normal(N, mean=7.0, std=1.75)
    return pos, scale, _unit(r.normal(4, N)), vsh, radius


def _scene(c, seed):
    """Planar tensors of an explicit scene and its member counts."""
    r = _Rng(seed)
    N, K, kind = c["cells"], c["K"], c["scene"]
    pos, scale, rot, vsh, radius = _cells(r, kind, N)
    t = {}
    if kind == "ragged":  # counts uniform over 0..K, a tenth full, a twentieth empty
        cnt = r.integers(0, K + 1, N)
        cnt = torch.where(r.uniform(N) < 0.1, torch.full_like(cnt, K), cnt)
        cnt = torch.where(r.uniform(N) < 0.05, torch.zeros_like(cnt), cnt)
        cnt[0] = K
        off = torch.zeros(N + 1, dtype=torch.int64, device=DEV)
        off[1:] = torch.cumsum(cnt, 0)
        t["cell_offsets"] = off.to(torch.int32)
        own = torch.repeat_interleave(torch.arange(N, device=DEV), cnt)
    else:
        own = torch.arange(N, device=DEV).repeat_interleave(K)
    M = int(own.numel())
    means = pos[:, own] + _rotate(rot[:, own], _ball(r, M) * scale[:, own])
    if kind == "large":
        scales = radius[own] * torch.exp(r.normal(3, M, mean=-1.5, std=0.4))
    else:
        scales = torch.exp(r.normal(3, M, mean=-5.5 if kind == "mid" else -4.5, std=0.4))
    opac = torch.sigmoid(r.normal(M) if kind in ("tiny", "ragged") else r.normal(M, mean=1.5, std=1.5))
    C = (c["degree"] + 1) ** 2
    sh = r.normal(C, 3, M, std=0.2)
    if kind in ("tiny", "ragged"):
        sh[0] = (r.uniform(3, M) - 0.5) * (2.0 * math.sqrt(math.pi))
    t.update(cell_pos=pos, cell_scale=scale, cell_rot=rot, cell_v_sh=vsh, means=means, scales=scales,
             rots=_unit(r.normal(4, M)), opacities=opac, sh=sh)
    return {k: v.contiguous() for k, v in t.items()}, M


def _camera(c):
    w, h, view = c["width"], c["height"], c["view"]
    if c.get("scene") == "large":
        return scenes.large_scene_cameras(2, w, h)[view % 40]
    return scenes.orbit_cameras(60, w, h)[view % 60]


def _device_scene(c, t, M):
    return DeviceScene(t, c["cells"], c["K"], 1, c["degree"], M if "cell_offsets" in t else None)


def _neural_scene(c, seed):
    """Tensors of a neural scene and the packed weights of its four decoders."""
    r = _Rng(seed)
    N, K, F, H = c["cells"], c["K"], c["F"], c["H"]
    pos, scale, rot, vsh, _ = _cells(r, "neural", N)
    t = dict(cell_pos=pos, cell_scale=scale, cell_rot=rot, cell_v_sh=vsh, features=r.normal(F, N),
             offsets=_ball(r, N * K) * 0.9)
    parts = []
    for a, bias in zip((1, 3, 3, 4), (1.5, 0.0, -1.25, None)):
        I, O = F + 4, K * a
        parts += [r.normal(I, H, std=1.0 / math.sqrt(I)), r.normal(H, std=0.1),
                  r.normal(H, O, std=0.5 / math.sqrt(H))]
        b2 = r.normal(O, std=0.3)
        if bias is None:  # quaternions: identity plus noise
            b2 = b2 + torch.tensor([2.0, 0.0, 0.0, 0.0], device=DEV).repeat(K)
        else:
            b2 = b2 + bias
        parts.append(b2)
    return {k: v.contiguous() for k, v in t.items()}, torch.cat([p.reshape(-1) for p in parts])


def _images(c, seed):
    """A rendered-like image (smooth and noisy parts) and its target."""
    r = _Rng(seed)
    C, H, W = c["channels"], c["height"], c["width"]
    low = r.uniform(1, C, max(2, H // 16), max(2, W // 16))
    y = torch.nn.functional.interpolate(low, size=(H, W), mode="bilinear", align_corners=True)[0]
    y = (y + r.normal(C, H, W, std=0.05)).clamp(0.0, 1.0).contiguous()
    return (y + r.normal(C, H, W, std=0.08)).contiguous(), y


LEAVES = ("cell_pos", "cell_v_sh", "means", "scales", "rots", "opacities", "sh")
PARAMS = ("cell_pos", "cell_scale", "cell_rot", "cell_v_sh", "means", "scales", "rots", "opacities", "sh")
SERVE_SIZES = ((640, 480), (1280, 720), (1920, 1080))


def _requests(c):
    """(scene, camera) of each request: two scenes, three sizes, orbit views."""
    out = []
    for i in range(c["requests"]):
        w, h = SERVE_SIZES[(i // 2) % 3]
        out.append((i % 2, scenes.orbit_cameras(12, w, h, step_deg=30.0)[(5 * i) % 12]))
    return out


def _mode(c):
    return dict(mode=c["mode"], tau=TAU) if c["mode"] == "lcwsr" else dict(mode=c["mode"])


def prepare(case, seed):
    c, kind = case, case["kind"]
    if kind == "frame":
        r = Renderer(0)
        t, M = _scene(c, seed)
        ds, cam = _device_scene(c, t, M), _camera(c)
        s = dict(kind=kind, r=r, ds=ds, cam=cam, out=r.alloc_image(cam), kw=_mode(c), check=c["check"])
        r.render(ds, cam, out=s["out"], **s["kw"])  # sizes the key buffers, as a program does before its loop
        return s
    if kind == "neural":
        r = Renderer(0)
        t, w = _neural_scene(c, seed)
        ns, cam = NeuralDeviceScene(t, c["cells"], c["K"], 1, c["F"], c["H"], w), _camera(c)
        s = dict(kind=kind, r=r, ds=ns, cam=cam, out=r.alloc_image(cam))
        r.render_neural(ns, cam, out=s["out"])
        return s
    if kind == "train":
        r = Renderer(0)
        t, M = _scene(c, seed)
        cam = _camera(c)
        g = _Rng(seed + 1000003)
        pert = dict(t)  # the target: a perturbed copy of the scene
        pert["means"] = t["means"] + g.normal(3, M, std=0.01)
        pert["opacities"] = torch.sigmoid(torch.logit(t["opacities"], eps=1e-6) + g.normal(M, std=0.3))
        target = r.render(_device_scene(c, pert, M), cam)["color"].clone()
        leaves = [t[k].requires_grad_(k in LEAVES) for k in PARAMS]
        return dict(kind=kind, r=r, cam=cam, leaves=leaves, target=target)
    if kind == "loss":
        x, y = _images(c, seed)
        return dict(kind=kind, r=Renderer(0), x=x, y=y, grad=c["grad"])
    if kind == "sort":
        g, n, bits = _Rng(seed), c["n"], c["bits"]
        keys = g.integers(-2 ** 63, 2 ** 63 - 1, n)
        if bits < 64:
            keys &= (1 << bits) - 1
        keys[n // 2:] = keys[: n - n // 2].clone()  # ties
        keys = keys[torch.randperm(n, device=DEV, generator=g.g)].contiguous()
        vals = torch.arange(n, device=DEV, dtype=torch.int32)
        return dict(kind=kind, r=Renderer(0), keys=keys, vals=vals, k=torch.empty_like(keys),
                    v=torch.empty_like(vals), bits=bits)
    assert kind == "serve"
    srv = Server(0, num_slots=4, use_graphs=True)
    ids = []
    for i, cells in enumerate((c["cells"], 5 * c["cells"])):
        sc = dict(kind="frame", scene="mid", cells=cells, K=c["K"], degree=3)
        t, M = _scene(sc, seed + 7919 * i)
        ids.append(srv.add_scene(_device_scene(sc, t, M)))
    torch.cuda.synchronize()
    reqs = [(ids[i], cam) for i, cam in _requests(c)]
    outs = [torch.empty((3, cam["height"], cam["width"]), device=DEV) for _, cam in reqs]
    s = dict(kind=kind, srv=srv, reqs=reqs, outs=outs)
    torch.cuda.synchronize()
    run(s)  # the server learns its key counts
    return s


def run(s):
    kind = s["kind"]
    if kind == "frame":
        return s["r"].render(s["ds"], s["cam"], out=s["out"], check=s["check"], **s["kw"])
    if kind == "neural":
        return s["r"].render_neural(s["ds"], s["cam"], out=s["out"], check=False)
    if kind == "train":
        for p in s["leaves"]:
            p.grad = None
        color, _ = DuplexRenderPlanar.apply(s["r"], s["cam"], {}, *s["leaves"])
        loss = L1SsimLoss.apply(s["r"], color, s["target"], LAMBDA)
        loss.backward()
        grads = {k: p.grad for k, p in zip(PARAMS, s["leaves"]) if p.requires_grad}
        return dict(loss=loss.detach(), color=color.detach(), grads=grads)
    if kind == "loss":
        loss, g = s["r"].loss_l1_ssim(s["x"], s["y"], LAMBDA, grad=s["grad"])
        return dict(loss=loss, grad=g) if s["grad"] else dict(loss=loss)
    if kind == "sort":
        s["k"].copy_(s["keys"])
        s["v"].copy_(s["vals"])
        s["r"].sort_pairs(s["k"], s["v"], s["bits"])
        return dict(keys=s["k"], vals=s["v"])
    srv = s["srv"]
    rids = [srv.submit(sid, cam, out=o) for (sid, cam), o in zip(s["reqs"], s["outs"])]
    for rid in rids:
        info, _ = srv.wait(rid, timeout=60.0)
        if info["state"] != capi.DGS_REQ_DONE:
            raise RuntimeError(f"request not served: {info}")
    return s["outs"]


# ------------------------------------------------------------------ work

def work(case):
    """Bytes of one pass: every scene value read once, every output written
    once.  Operations: the projection of each Gaussian (~400 with its colour),
    and per pixel the ~30 members that reach it (as on the clustered scene) at
    ~30 operations each for a frame, three times that with its gradient."""
    c, kind = case, case["kind"]
    if kind == "sort":
        return dict(bytes=24.0 * c["n"], flops=0.0)
    if kind == "loss":
        n = c["channels"] * c["width"] * c["height"]
        return dict(bytes=n * (12.0 if c["grad"] else 8.0), flops=n * (300.0 if c["grad"] else 170.0))
    if kind == "serve":
        b = f = 0.0
        for i, cam in _requests(c):
            w = work(dict(kind="frame", scene="mid", cells=c["cells"] * (1, 5)[i], K=c["K"], degree=3,
                          width=cam["width"], height=cam["height"]))
            px = cam["width"] * cam["height"]
            b, f = b + w["bytes"] - 12.0 * px, f + w["flops"]
        return dict(bytes=b, flops=f)
    px, N = c["width"] * c["height"], c["cells"]
    M = N * c["K"] * (0.55 if c.get("scene") == "ragged" else 1.0)
    cell = N * 4.0 * (3 + 3 + 4 + 4)
    if kind == "neural":
        macs = sum((c["F"] + 4) * c["H"] + c["H"] * c["K"] * a for a in (1, 3, 3, 4))
        return dict(bytes=cell + 4.0 * N * c["F"] + 12.0 * M + 24.0 * px, flops=2.0 * N * macs + 200.0 * M + 900.0 * px)
    gauss = M * 4.0 * (3 + 3 + 4 + 1 + 3 * (c["degree"] + 1) ** 2)
    if kind == "train":
        return dict(bytes=2.0 * (cell + gauss) + 28.0 * px, flops=1200.0 * M + 2700.0 * px + 900.0 * px)
    return dict(bytes=cell + gauss + 24.0 * px, flops=400.0 * M + 900.0 * px)


# ------------------------------------------------------------------ 64-bit values

ALPHA_MIN, ALPHA_MAX, EPS, DELTA, TILE = 1.0 / 255.0, 0.99, 1e-4, 0.3, 16


def _sh(c, d):
    """Real spherical harmonics of direction d dotted with c [C, ..., n]."""
    x, y, z = d
    xx, yy, zz = x * x, y * y, z * z
    k = lambda a, b=1.0: math.sqrt(a / math.pi) * b  # noqa: E731
    Y = [k(1, 0.5) * torch.ones_like(x),
         -k(0.75) * y, k(0.75) * z, -k(0.75) * x,
         k(15, 0.5) * x * y, -k(15, 0.5) * y * z, k(5, 0.25) * (2 * zz - xx - yy), -k(15, 0.5) * x * z,
         k(15, 0.25) * (xx - yy),
         -k(70, 0.125) * y * (3 * xx - yy), k(105, 0.5) * x * y * z, -k(42, 0.125) * y * (4 * zz - xx - yy),
         k(7, 0.25) * z * (2 * zz - 3 * xx - 3 * yy), -k(42, 0.125) * x * (4 * zz - xx - yy),
         k(105, 0.25) * z * (xx - yy), -k(70, 0.125) * x * (xx - 3 * yy)]
    return sum(c[j] * Y[j] for j in range(c.shape[0]))


def _project(cam, dt, pos, scale, rot):
    """Camera-space position, screen covariance (xx, xy, yy) and screen
    position, in type dt, by one fixed order of operations."""
    V = torch.tensor(np.asarray(cam["viewmat"], np.float32), device=DEV).to(dt)
    W, H = cam["width"], cam["height"]
    f32 = lambda v: torch.tensor(v, dtype=torch.float32, device=DEV).to(dt)  # noqa: E731
    fx, fy, cx, cy = f32(cam["fx"]), f32(cam["fy"]), f32(cam["cx"]), f32(cam["cy"])
    R = V[:3, :3]
    p, s, q = pos.to(dt), scale.to(dt), rot.to(dt)
    t = [((R[i, 0] * p[0] + R[i, 1] * p[1]) + R[i, 2] * p[2]) + V[i, 3] for i in range(3)]
    n = torch.sqrt(((q[0] * q[0] + q[1] * q[1]) + q[2] * q[2]) + q[3] * q[3])
    w, x, y, z = (q[i] / n for i in range(4))
    Q = [[1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y)],
         [2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x)],
         [2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)]]
    M = [[Q[i][j] * s[j] for j in range(3)] for i in range(3)]
    S = [[(M[i][0] * M[j][0] + M[i][1] * M[j][1]) + M[i][2] * M[j][2] for j in range(3)] for i in range(3)]
    limx, limy = f32(1.3) * ((0.5 * W) / fx), f32(1.3) * ((0.5 * H) / fy)
    tx = torch.minimum(limx, torch.maximum(-limx, t[0] / t[2])) * t[2]
    ty = torch.minimum(limy, torch.maximum(-limy, t[1] / t[2])) * t[2]
    z2 = t[2] * t[2]
    j00, j02, j11, j12 = fx / t[2], -(fx * tx) / z2, fy / t[2], -(fy * ty) / z2
    m = [[j00 * R[0, j] + j02 * R[2, j] for j in range(3)], [j11 * R[1, j] + j12 * R[2, j] for j in range(3)]]
    u = [[(m[r][0] * S[0][j] + m[r][1] * S[1][j]) + m[r][2] * S[2][j] for j in range(3)] for r in range(2)]
    dot = lambda a, b: (a[0] * b[0] + a[1] * b[1]) + a[2] * b[2]  # noqa: E731
    return t, (dot(u[0], m[0]), dot(u[0], m[1]), dot(u[1], m[1])), (fx * (t[0] / t[2]) + cx, fy * (t[1] / t[2]) + cy)


def _rect(cam, ux, uy, hx, hy, ok):
    """Pixel rectangle x0, x1, y0, y1 (int64) and whether it holds a pixel."""
    x0, x1 = torch.ceil((ux - hx) - 0.5), torch.floor((ux + hx) - 0.5)
    y0, y1 = torch.ceil((uy - hy) - 0.5), torch.floor((uy + hy) - 0.5)
    ok = ok & (x0 <= x1) & (y0 <= y1)
    x0, x1 = x0.clamp(min=0), x1.clamp(max=cam["width"] - 1)
    y0, y1 = y0.clamp(min=0), y1.clamp(max=cam["height"] - 1)
    ok = ok & (x0 <= x1) & (y0 <= y1)
    return [torch.where(ok, v, torch.zeros_like(v)).to(torch.int64) for v in (x0, x1, y0, y1)], ok


def _direction(cam, p):
    V = torch.tensor(np.asarray(cam["viewmat"], np.float32), device=DEV).double()
    o = -(V[:3, :3].t() @ V[:3, 3])
    d = p - o[:, None]
    return d / torch.sqrt((d * d).sum(0))


def _exact_frame(t, cam, K, mode="duplex", offsets=None, color=None):
    """The frame in binary64 from planar tensors t: boxes and tile lists from
    a binary32 projection, everything else from t's binary64 values (with
    gradients, where t asks for them).  Returns color, D, T."""
    f32, f64 = torch.float32, torch.float64
    W, H = cam["width"], cam["height"]
    TX, TY = (W + TILE - 1) // TILE, (H + TILE - 1) // TILE
    znear = float(np.float32(cam.get("z_near", 0.2)))
    t64 = {k: v.to(f64) for k, v in t.items() if k != "cell_offsets"}
    with torch.no_grad():
        gt, gcov, gu = _project(cam, f32, t["means"].detach(), t["scales"].detach(), t["rots"].detach())
        dl = torch.tensor(DELTA, dtype=f32, device=DEV)
        gok = (t["opacities"].detach() > 0) & (gt[2] > znear)
        grect, gok = _rect(cam, gu[0], gu[1], 3.0 * torch.sqrt(gcov[0] + dl), 3.0 * torch.sqrt(gcov[2] + dl), gok)
        M = gok.numel()
        if mode == "alpha":
            prect, pok, depth, K = grect, gok, gt[2], 1
            first, count = torch.arange(M, device=DEV), torch.ones(M, dtype=torch.int64, device=DEV)
        else:
            ct, ccov, cu = _project(cam, f32, t["cell_pos"].detach(), t["cell_scale"].detach(), t["cell_rot"].detach())
            pad = 3.0 * torch.sqrt(dl)
            prect, pok = _rect(cam, cu[0], cu[1], torch.sqrt(ccov[0]) + pad, torch.sqrt(ccov[2]) + pad, ct[2] > znear)
            depth, N = ct[2], pok.numel()
            if offsets is not None:
                first = offsets[:-1].to(torch.int64)
                count = offsets[1:].to(torch.int64) - first
            else:
                first = torch.arange(N, device=DEV) * K
                count = torch.full_like(first, K)
        # tile lists in (tile, depth, id) order
        ids = torch.nonzero(pok)[:, 0]
        tx0, tx1, ty0, ty1 = (v[ids] // TILE for v in prect)
        nx = tx1 - tx0 + 1
        nt = nx * (ty1 - ty0 + 1)
        rep = torch.repeat_interleave(torch.arange(ids.numel(), device=DEV), nt)
        j = torch.arange(rep.numel(), device=DEV) - (torch.cumsum(nt, 0) - nt)[rep]
        tile = (ty0[rep] + j // nx[rep]) * TX + tx0[rep] + j % nx[rep]
        bits = depth.view(torch.int32).to(torch.int64)[ids][rep]
        key, perm = torch.sort((tile << 32) | bits, stable=True)
        lists, tile = ids[rep][perm], key >> 32
        start = torch.searchsorted(tile, torch.arange(TX * TY, device=DEV))
        length = torch.searchsorted(tile, torch.arange(TX * TY, device=DEV), right=True) - start
    # continuous part
    _, cov, u = _project(cam, f64, t64["means"], t64["scales"], t64["rots"])
    a, b, c = cov[0] + float(np.float32(DELTA)), cov[1], cov[2] + float(np.float32(DELTA))
    det = a * c - b * b
    rgb = color if color is not None else torch.relu(0.5 + _sh(t64["sh"], _direction(cam, t64["means"])))
    attr = torch.stack([u[0], u[1], c / det, -b / det, a / det, t64["opacities"], rgb[0], rgb[1], rgb[2]], 1)
    attr = torch.where(gok[:, None], attr, torch.zeros_like(attr))
    box = torch.stack([torch.where(gok, grect[0], torch.full_like(grect[0], 1 << 40))] + grect[1:], 1)
    v = torch.sigmoid(_sh(t64["cell_v_sh"], _direction(cam, t64["cell_pos"]))) if mode != "alpha" else None
    if mode == "lcwsr":
        v = v * torch.relu(1.0 - depth.to(f64) / TAU)
    pix = torch.arange(TILE * TILE, device=DEV)
    order = torch.argsort(length, descending=True)
    order = order[length[order] > 0]
    n = order.numel()
    px = (order % TX)[:, None] * TILE + pix % TILE
    py = (order // TX)[:, None] * TILE + pix // TILE
    grad = attr.requires_grad
    state = torch.zeros(5, n, TILE * TILE, dtype=f64, device=DEV)  # N or C (3), D, T
    state[4] = 1.0
    ln = length[order].tolist()
    act = torch.arange(n, device=DEV)  # tiles still walked (a prefix order in list length, thinned as they end)
    cur, done, kk = state, [], torch.arange(K, device=DEV)
    p, live, at = 0, n, act
    while True:
        while live and ln[live - 1] <= p:
            live -= 1
        if p % 32 == 0 or live < at.numel():
            keep = at < live
            if not grad and mode != "lcwsr":
                keep &= (cur[4] >= EPS).any(1)
            if not bool(keep.all()):
                done.append((at[~keep], cur[:, ~keep]))
                at, cur = at[keep], cur[:, keep]
        if at.numel() == 0:
            break
        cell = lists[start[order[at]] + p]
        m = (first[cell][:, None] + kk).clamp(max=M - 1)
        have = kk < count[cell][:, None]
        e, bx = attr[m], box[m]
        X, Y = px[at][:, None, :], py[at][:, None, :]
        dx, dy = X + 0.5 - e[..., 0:1], Y + 0.5 - e[..., 1:2]
        inb = have[..., None] & (X >= bx[..., 0:1]) & (X <= bx[..., 1:2]) & (Y >= bx[..., 2:3]) & (Y <= bx[..., 3:4])
        al = e[..., 5:6] * torch.exp(-0.5 * (e[..., 2:3] * dx * dx + e[..., 4:5] * dy * dy) - e[..., 3:4] * dx * dy)
        T = cur[4]
        on = inb & (al.detach() >= ALPHA_MIN)
        if mode != "lcwsr":
            on = on & (T.detach() >= EPS)[:, None, :]
        al = torch.where(on, al.clamp(max=ALPHA_MAX), torch.zeros_like(al))
        if mode == "alpha":
            w = T * al[:, 0]
            cur = torch.stack([cur[q] + w * e[:, 0, 6 + q, None] for q in range(3)] + [cur[3] + w, T - w])
        else:
            vc = v[cell][:, None]
            w = vc if mode == "lcwsr" else vc * T
            P = torch.prod(1.0 - vc[..., None] * al, 1) if mode != "lcwsr" else 1.0
            cur = torch.stack([cur[q] + w * (al * e[..., 6 + q:7 + q]).sum(1) for q in range(3)]
                              + [cur[3] + w * al.sum(1), T * P])
        p += 1
    full = torch.zeros(5, TX * TY, TILE * TILE, dtype=f64, device=DEV)
    full[4] = 1.0
    if done:
        full = full.index_copy(1, order[torch.cat([i for i, _ in done])], torch.cat([s for _, s in done], 1))
    img = full.reshape(5, TY, TX, TILE, TILE).permute(0, 1, 3, 2, 4).reshape(5, TY * TILE, TX * TILE)[:, :H, :W]
    if mode == "alpha":
        return img[:3], 1.0 - img[4], img[4]
    D = img[3]
    return torch.where(D > 0, img[:3] / torch.where(D > 0, D, torch.ones_like(D)), torch.zeros_like(img[:3])), D, img[4]


def _exact_loss(x, y):
    """The training loss of images x, y [C, H, W] in binary64."""
    g = torch.exp(-0.5 * ((torch.arange(11, device=DEV, dtype=torch.float64) - 5) / 1.5) ** 2)
    g = g / g.sum()

    def blur(a):
        a = torch.nn.functional.pad(a, (5, 5, 5, 5))
        a = sum(g[k] * a[:, :, k:a.shape[2] - 10 + k] for k in range(11))
        return sum(g[k] * a[:, k:a.shape[1] - 10 + k] for k in range(11))

    mx, my = blur(x), blur(y)
    sxx, syy, sxy = blur(x * x) - mx * mx, blur(y * y) - my * my, blur(x * y) - mx * my
    c1, c2 = 0.01 ** 2, 0.03 ** 2
    ssim = (2 * mx * my + c1) * (2 * sxy + c2) / ((mx * mx + my * my + c1) * (sxx + syy + c2))
    return (1 - LAMBDA) * (x - y).abs().mean() + LAMBDA * (1 - ssim.mean())


def _exact_decode(c, t, w, cam):
    """Decoded Gaussians of a neural scene in binary64, planar, and colours."""
    N, K, F, H = c["cells"], c["K"], c["F"], c["H"]
    t = {k: v.double() for k, v in t.items()}
    w = w.double()
    V = torch.tensor(np.asarray(cam["viewmat"], np.float32), device=DEV).double()
    e = t["cell_pos"] - (-(V[:3, :3].t() @ V[:3, 3]))[:, None]
    dist = torch.sqrt((e * e).sum(0, keepdim=True))
    x = torch.cat([t["features"], dist, e / dist]).t()
    outs, at = [], 0
    for a in (1, 3, 3, 4):
        I, O = F + 4, K * a
        take = lambda n, sh: w[at:at + n].reshape(sh)  # noqa: E731
        W1 = take(I * H, (I, H)); at += I * H  # noqa: E702
        b1 = take(H, (H,)); at += H  # noqa: E702
        W2 = take(H * O, (H, O)); at += H * O  # noqa: E702
        b2 = take(O, (O,)); at += O  # noqa: E702
        outs.append((torch.relu(x @ W1 + b1) @ W2 + b2).reshape(N * K, a).t())
    own = torch.arange(N, device=DEV).repeat_interleave(K)
    off, S = t["offsets"], t["cell_scale"][:, own]
    means = t["cell_pos"][:, own] + _rotate(t["cell_rot"][:, own], off * S)
    lim = 1.0 - torch.sqrt((off * off).sum(0))
    scales = torch.relu(torch.minimum(torch.sigmoid(outs[2]), lim)) * S
    g = dict(t, means=means, scales=scales, rots=outs[3], opacities=torch.tanh(outs[0][0]))
    return g, torch.sigmoid(outs[1])


def exact(case, seed):
    c, kind = case, case["kind"]
    if kind in ("sort", "serve"):  # whole numbers; frames that the frame cases hold, in a dozen
        return None
    if kind == "loss":
        x, y = _images(c, seed)
        x, y = x.double().requires_grad_(c["grad"]), y.double()
        loss = _exact_loss(x, y)
        if not c["grad"]:
            return dict(loss=loss)
        loss.backward()
        return dict(loss=loss.detach(), grad=x.grad)
    cam = _camera(c)
    if kind == "neural":
        t, w = _neural_scene(c, seed)
        g, col = _exact_decode(c, t, w, cam)
        color, D, T = _exact_frame(g, cam, c["K"], color=col)
        return dict(color=color, D=D, T=T, last=None)
    t, M = _scene(c, seed)
    if kind == "frame":
        color, D, T = _exact_frame(t, cam, c["K"], c["mode"], t.get("cell_offsets"))
        return dict(color=color, D=D, T=torch.ones_like(T) if c["mode"] == "lcwsr" else T, last=None)
    g = _Rng(seed + 1000003)
    pert = dict(t)
    pert["means"] = t["means"] + g.normal(3, M, std=0.01)
    pert["opacities"] = torch.sigmoid(torch.logit(t["opacities"], eps=1e-6) + g.normal(M, std=0.3))
    target = _exact_frame(pert, cam, c["K"])[0]
    # the graph of every list step is kept: small frames only
    small = c["width"] * c["height"] <= 1 << 17 and c["cells"] * c["K"] <= 1 << 15
    p = {k: v.double().requires_grad_(small and k in LEAVES) for k, v in t.items()}
    color, _, _ = _exact_frame(p, cam, c["K"])
    loss = _exact_loss(color, target)
    if small:
        loss.backward()
    grads = {k: p[k].grad if small else None for k in LEAVES}
    return dict(loss=loss.detach(), color=color.detach(), grads=grads)

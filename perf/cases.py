"""The framework's work as a user has it do, case by case, for timing and for comparing outputs.

Each case is a dict of plain values; ``kind`` names the path:

* ``chain``: a planned chain of the fixed stages (the Harris chains, the gradient chain) on a
  resident clip, through ``Plan.run`` with buffers the program keeps.  The feature points come in
  no fixed order, so a pass returns their count beside the whole output video;
* ``generic``: the same with plan-time stages (window stages, point stages, IIR filters, stencils
  over several frames), on the default engine or on generated kernels (``engine="jit"``);
* ``batch``: many clips of different sizes through one ``run_batch`` call;
* ``track``: Kalman tracking of a clip's feature points (``fz_track_points``);
* ``mlp``: the cost network: one training step (loss, gradient, Adam) or a prediction.

``listed`` gives the fixed cases, ``draw`` one more of the same ranges, ``prepare`` what a program
holds before the call (made on the GPU from the seed alone), ``run`` one pass, ``work`` the bytes
and operations a pass cannot do without, ``exact`` the outputs in 64 bits from plain torch and numpy.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1509_04394_amd import fz, synth

# Frame sizes of the repository's workloads, and ragged ones (tile and strip
# remainders, widths that are no multiple of 4, frames narrower than 128).
SIZES = [(192, 432), (320, 240), (640, 480), (800, 600)]
RAGGED = [(641, 479), (333, 251), (799, 601), (203, 77), (150, 70), (96, 80), (255, 129), (510, 382)]


def listed():
    return [
        # the headline: a whole high-speed RGB clip, every stage fused
        dict(name="harris rgb 800x600x1000", kind="chain", chain="rgb_harris", W=800, H=600, T=1000, partition="optimal"),
        # the narrow gray clips of the paper's camera
        dict(name="harris gray 192x432x600", kind="chain", chain="harris", W=192, H=432, T=600, partition="optimal"),
        # gradient maps in f32 of a short clip
        dict(name="gradient 192x432x64", kind="chain", chain="grad", W=192, H=432, T=64, partition="optimal"),
        # a live feed handed over a few frames at a time: latency
        dict(name="harris rgb 320x240x4", kind="chain", chain="rgb_harris", W=320, H=240, T=4, partition="optimal"),
        # every stage as its own kernel (a program that keeps or inspects the intermediates), odd sizes
        dict(name="harris unfused 641x479x75", kind="chain", chain="harris", W=641, H=479, T=75, partition="unfused"),
        # a short user-defined chain on the default engine, as in the quick start
        dict(name="generic 800x600x64", kind="generic", chain="generic3", W=800, H=600, T=64, dtype="u8", engine="auto"),
        # a long random chain of the learned-price workload, fed with f32 frames
        dict(name="random f32 320x240x64", kind="generic", chain="random", chain_seed=9505, W=320, H=240, T=64,
             dtype="f32", engine="auto"),
        # stencils over several frames on the default engine, odd frame size
        dict(name="lookback 333x251x200", kind="generic", chain="spatio", W=333, H=251, T=200, dtype="u8", engine="auto"),
        # the paper's five kernels over a whole clip, generated kernels
        dict(name="paper5 jit 800x600x1000", kind="generic", chain="paper5", W=800, H=600, T=1000, dtype="u8",
             engine="jit"),
        # an archive of clips through the persistent launch
        dict(name="batch 16 clips", kind="batch", clips=16, clip_seed=4, t_lo=50, t_hi=400),
        # tracks of a clip with about as many points per frame as the headline clip gives
        dict(name="track 1000 frames", kind="track", W=800, H=600, T=1000, objects=40, clutter=1.0),
        # a training step of the cost network at the trainer's batch size
        dict(name="mlp step 8192", kind="mlp", n=8192, features=20, predict=False),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _frame(rng):
    """A frame size: one of the workloads', a ragged one, or any in their range."""
    k = rng.randrange(3)
    if k == 0:
        return rng.choice(SIZES)
    if k == 1:
        return rng.choice(RAGGED)
    return _log_int(rng, 96, 800), _log_int(rng, 64, 600)


def draw(rng):
    kind = rng.choice(["chain", "chain", "chain", "generic", "generic", "generic", "batch", "track", "mlp"])
    W, H = _frame(rng)
    if kind == "chain":
        partition = rng.choice(["optimal", "optimal", "optimal", "unfused"])
        chain = rng.choice(["rgb_harris", "harris", "grad"])
        most = 480e6 if partition == "optimal" and chain != "grad" else 60e6
        T = max(2, min(_log_int(rng, 2, 1000), int(most / (W * H))))
        return dict(kind=kind, chain=chain, W=W, H=H, T=T, partition=partition)
    if kind == "generic":
        chain = rng.choice(["generic3", "paper5", "spatio", "random", "random"])
        engine = rng.choice(["auto", "auto", "jit"])
        T = max(2, min(_log_int(rng, 4, 600), int(60e6 / (W * H))))
        c = dict(kind=kind, chain=chain, W=W, H=H, T=T, dtype=rng.choice(["u8", "u8", "f32"]), engine=engine)
        if chain == "random":
            c["chain_seed"] = _random_seed(rng)
        return c
    if kind == "batch":
        return dict(kind=kind, clips=rng.randint(2, 16), clip_seed=rng.randrange(1, 1 << 20), t_lo=8,
                    t_hi=_log_int(rng, 40, 200))
    if kind == "track":
        return dict(kind=kind, W=W, H=H, T=_log_int(rng, 16, 1000), objects=_log_int(rng, 4, 90),
                    clutter=round(rng.uniform(0.0, 4.0), 2))
    return dict(kind="mlp", n=_log_int(rng, 64, 65536), features=rng.choice([20, 20, 7, 32]),
                predict=rng.random() < 0.3)


# ---------------------------------------------------------------- chains
def _magnitude(spec):
    """A bound on the values a generic chain can reach from u8 input."""
    m, top = 255.0, 255.0
    for st in spec:
        if st[0] == "point":
            k, a, b = st[1], abs(st[2]), abs(st[3])
            m = {"affine": a * m + b, "abs": m, "square": m * m, "sqrtabs": math.sqrt(m), "clamp": max(a, b)}[k]
        elif st[0] == "box":
            m *= (2 * st[1] + 1) * (2 * st[2] + 1)
        top = max(top, m)
    return top


def _random_seed(rng):
    """A random chain of the repository's test split whose values stay in single precision's range,
    without a clamp (after a window sum most of them leave one constant)."""
    while True:
        s = rng.randrange(9500, 10000)
        spec = synth.random_chain(s)
        if _magnitude(spec) < 1e15 and not any(st[1] == "clamp" for st in spec if st[0] == "point"):
            return s


def _spec(case):
    name = case["chain"]
    if name == "generic3":  # 3x3 binomial, magnitude, 3x3 window sum
        return [("stencil", 1, 1, (np.outer([1, 2, 1], [1, 2, 1]) / 16.0).astype(np.float32)),
                ("point", "abs", 0.0, 0.0), ("box", 1, 1)]
    if name == "paper5":  # IIR, 5x5 Gaussian, horizontal Sobel, magnitude, clamp
        g = np.exp(-np.arange(-2, 3) ** 2 / 2.0)
        g5 = (np.outer(g, g) / np.outer(g, g).sum()).astype(np.float32)
        sx = np.array([[-1, 0, 1], [-2, 0, 2], [-1, 0, 1]], np.float32)
        return [("iir", float(np.float32(0.3))), ("stencil", 2, 2, g5), ("stencil", 1, 1, sx),
                ("point", "abs", 0.0, 0.0), ("point", "clamp", 0.0, 200.0)]
    if name == "spatio":  # stencils over three and two frames
        w33 = ((np.arange(27, dtype=np.float32).reshape(3, 3, 3) % 5 + 1.0) / 60.0).astype(np.float32)
        w253 = (((np.arange(30, dtype=np.float32).reshape(2, 3, 5) % 7) - 3.0) / 40.0).astype(np.float32)
        return [("point", "affine", 0.5, 1.0), ("stencil", 1, 1, w33), ("box", 1, 1), ("stencil", 2, 1, w253),
                ("point", "sqrtabs", 0.0, 0.0)]
    if name == "random":
        return synth.random_chain(case["chain_seed"])
    return {"rgb_harris": fz.RGB_HARRIS_CHAIN, "harris": fz.HARRIS_CHAIN, "grad": fz.GRAD_CHAIN}[name]


# ---------------------------------------------------------------- inputs
def _video(W, H, T, seed, rgb=False):
    """u8 high-speed video on the GPU, of the character of ``synth.video``: a smooth static
    background in [40, 200] per channel, 20 moving blobs (sigma 3, +60) on the frame torus,
    N(0, 4^2) noise per pixel and channel."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    r = np.random.default_rng(seed)
    C = 3 if rgb else 1
    grid = torch.tensor(r.uniform(0.0, 1.0, (1, C, 4, 6)), dtype=torch.float32, device="cuda")
    bg = torch.nn.functional.interpolate(grid, size=(H, W), mode="bicubic", align_corners=True)[0]
    lo, hi = bg.amin((1, 2), keepdim=True), bg.amax((1, 2), keepdim=True)
    bg = ((bg - lo) / (hi - lo).clamp_min(1e-12) * 160.0 + 40.0).permute(1, 2, 0)  # [H][W][C]
    n, t = 20, np.arange(T)[:, None]
    speed, ang = r.uniform(0, 1, n), r.uniform(0, 2 * np.pi, n)

    def centres(size, v):
        return np.mod(r.uniform(0, size, n) + v * t + r.uniform(2, 10, n) *
                      np.sin(r.uniform(0.02, 0.2, n) * t + r.uniform(0, 2 * np.pi, n)), size)

    def profile(size, c):  # [T][n][size]: the blobs' profile along one axis, wrapped
        c = torch.tensor(c, dtype=torch.float32, device="cuda")[:, :, None]
        d = (torch.arange(size, device="cuda", dtype=torch.float32) - c).abs()
        d = torch.minimum(d, size - d)
        return torch.exp(-d * d / 18.0)

    cx, cy = centres(W, speed * np.cos(ang)), centres(H, speed * np.sin(ang))
    out = torch.empty((T, H, W, C), dtype=torch.uint8, device="cuda")
    step = max(1, int(60e6 / (W * H * C)))
    for k in range(0, T, step):
        gx, gy = profile(W, cx[k:k + step]), profile(H, cy[k:k + step])
        f = torch.zeros((gx.shape[0], H, W), device="cuda")
        for i in range(n):  # one blob after another: the sums come in one order
            f.addcmul_(gy[:, i, :, None], gx[:, i, None, :], value=60.0)
        f = f[..., None] + bg
        f += torch.randn(f.shape, generator=g, device="cuda").mul_(4.0)
        out[k:k + step] = f.round_().clamp_(0, 255).to(torch.uint8)
    return out if rgb else out[..., 0].contiguous()


def _points(case, seed):
    """Feature points (t, y, x) of moving objects and clutter, each pixel at most once a frame, shuffled."""
    r = np.random.default_rng(seed)
    W, H, T, n = case["W"], case["H"], case["T"], case["objects"]
    t = np.arange(T)[:, None]
    speed, ang = r.uniform(0, 1, n), r.uniform(0, 2 * np.pi, n)
    size = np.array([W, H])
    p = (r.uniform(0, size, (n, 2)) + np.stack([speed * np.cos(ang), speed * np.sin(ang)], 1) * t[:, :, None] +
         r.uniform(2, 10, (n, 2)) * np.sin(r.uniform(0.02, 0.2, (n, 2)) * t[:, :, None] + r.uniform(0, 6.28, (n, 2))))
    p = np.mod(np.rint(p + r.normal(0, 0.4, p.shape)), size).astype(np.int64)
    seen = r.uniform(size=(T, n)) < 0.93
    frame = np.broadcast_to(t, (T, n))[seen]
    extra = int(case["clutter"] * T)
    q = np.concatenate([np.stack([frame, p[seen][:, 1], p[seen][:, 0]], 1),
                        np.stack([r.integers(0, T, extra), r.integers(0, H, extra), r.integers(0, W, extra)], 1)])
    q = np.unique(q, axis=0)
    return q[r.permutation(len(q))].astype(np.int32)


def _record_capacity(case):
    """Room for a record a point and one a missed frame after it."""
    return int(case["T"] * (case["objects"] + case["clutter"]) * 4) + 64


def _mlp_state(case, seed):
    """Parameters, moments and a batch as in the middle of a training run."""
    r = np.random.default_rng(seed)
    F, n, h = case["features"], case["n"], 64
    f32 = lambda v: np.ascontiguousarray(v, np.float32)
    prm = f32(np.concatenate([r.normal(0, math.sqrt(2.0 / F), h * F), r.normal(0, 0.1, h),
                              r.normal(0, math.sqrt(2.0 / h), h * h), r.normal(0, 0.1, h),
                              r.normal(0, math.sqrt(1.0 / h), h), [5.0]]))
    x = f32(r.normal(0.5, 1.0, (n, F)))
    t = f32(5.0 + x @ r.normal(0, 0.4, F) + r.normal(0, 0.1, n))
    m = f32(r.normal(0, 1e-2, prm.size))
    v = f32(np.abs(r.normal(0, 1e-2, prm.size)) ** 2 + 1e-6)
    return prm, x, t, m, v


# ---------------------------------------------------------------- prepare and run
def prepare(case, seed):
    s = dict(kind=case["kind"], stream=torch.cuda.current_stream().cuda_stream)
    kind = case["kind"]
    if kind == "chain":
        W, H, T = case["W"], case["H"], case["T"]
        s["plan"] = fz.Plan(_spec(case), W, H, T, partition=case["partition"])
        s["x"] = _video(W, H, T, seed, rgb=case["chain"] == "rgb_harris")
        s["bufs"] = s["plan"].alloc(point_capacity=1 << 18)
    elif kind == "generic":
        W, H, T = case["W"], case["H"], case["T"]
        s["plan"] = fz.Plan(_spec(case), W, H, T, engine=case["engine"], in_dtype=case["dtype"])
        x = _video(W, H, T, seed)
        s["x"] = x if case["dtype"] == "u8" else x.to(torch.float32)[None].contiguous()
        s["bufs"] = s["plan"].alloc()
    elif kind == "batch":
        plan = fz.Plan(fz.HARRIS_CHAIN, 800, 600, 1000)
        s["plan"], s["keep"], s["clips"] = plan, [], []
        for i, (W, H, T) in enumerate(synth.batch_shapes(case["clip_seed"], case["clips"], case["t_lo"], case["t_hi"])):
            x = _video(W, H, T, seed * 64 + i)
            out = torch.empty((T, H, W), dtype=torch.uint8, device="cuda")
            pts = torch.empty((1 << 16, 4), dtype=torch.int32, device="cuda")
            cnt = torch.zeros((1,), dtype=torch.int32, device="cuda")
            s["keep"].append((x, out, pts, cnt))
            s["clips"].append(fz.make_clip(x, out, pts, cnt, plan=plan))
        need = fz.fz_batch_workspace_bytes(plan.handle, s["clips"])
        s["ws"] = torch.empty((max(need, 1),), dtype=torch.uint8, device="cuda")
    elif kind == "track":
        p = _points(case, seed)
        pts = np.zeros((len(p), 4), np.int32)
        pts[:, :3] = p
        o = fz.track_opts()
        cap = _record_capacity(case)
        s.update(points=torch.tensor(pts, device="cuda"), count=torch.tensor([len(p)], dtype=torch.int32, device="cuda"),
                 opts=o, T=case["T"], records=torch.zeros((cap, 12), dtype=torch.int32, device="cuda"),
                 n_records=torch.zeros((2,), dtype=torch.int32, device="cuda"),
                 ws=torch.empty((fz.fz_track_workspace_bytes(case["T"], len(p), o),), dtype=torch.uint8, device="cuda"))
    else:
        prm, x, t, m, v = (torch.tensor(a, device="cuda") for a in _mlp_state(case, seed))
        F, n = case["features"], case["n"]
        s.update(F=F, n=n, predict=case["predict"], prm=prm, x=x, t=t, m=m, v=v, step=100,
                 y=torch.empty(n, device="cuda"), grad=torch.empty_like(prm), loss=torch.empty(1, device="cuda"),
                 ws=torch.empty(fz.fz_mlp_workspace_bytes(F, n), dtype=torch.uint8, device="cuda"))
    return s


def run(s):
    kind = s["kind"]
    if kind in ("chain", "generic"):
        out, pts, cnt, ws = s["bufs"]
        s["plan"].run(s["x"], out, pts, cnt, ws)
        return [out] if cnt is None else [out, cnt]
    if kind == "batch":
        fz.run_batch(s["plan"], s["clips"], s["ws"])
        return [[out, cnt] for _, out, _, cnt in s["keep"]]
    if kind == "track":
        r = s["records"]
        fz.fz_track_points(s["points"].data_ptr(), s["count"].data_ptr(), s["points"].shape[0], s["T"], s["opts"],
                           r.data_ptr(), s["n_records"].data_ptr(), r.shape[0], s["ws"].data_ptr(), s["ws"].numel(),
                           s["stream"])
        return [s["n_records"], r[:, :3], r.view(torch.float64)[:, 2:]]  # t, id, status; x, y, vx, vy
    if s["predict"]:
        fz.fz_mlp_forward(s["prm"].data_ptr(), s["F"], s["x"].data_ptr(), s["n"], s["y"].data_ptr(), s["stream"])
        return [s["y"]]
    P = s["prm"].numel()
    fz.fz_mlp_loss_grad(s["prm"].data_ptr(), s["F"], s["x"].data_ptr(), s["t"].data_ptr(), s["n"], s["grad"].data_ptr(),
                        s["loss"].data_ptr(), s["ws"].data_ptr(), s["ws"].numel(), s["stream"])
    fz.fz_mlp_adam_step(s["prm"].data_ptr(), s["grad"].data_ptr(), s["m"].data_ptr(), s["v"].data_ptr(), P, s["step"],
                        3e-3, 0.9, 0.999, 1e-8, s["stream"])
    s["step"] += 1
    return [s["loss"], s["grad"], s["prm"], s["m"], s["v"]]


# ---------------------------------------------------------------- work
# operations per output pixel of the fixed stages, every intermediate formed once, separable passes
OPS = {"rgb2gray": 9, "gauss5": 10, "sobel3": 6, "gradmag": 3, "products": 3, "boxsum5": 12, "harris": 5, "threshold": 2,
       "nms3": 7, "framediff": 2}


def _stage_ops(st):
    if st[0] == "point":
        return 2 if st[1] == "clamp" else 1
    if st[0] == "iir":
        return 2
    n = (2 * st[1] + 1) * (2 * st[2] + 1)
    return 2 * np.asarray(st[3]).size if st[0] == "stencil" else n - 1


def work(case):
    kind = case["kind"]
    if kind in ("chain", "generic"):
        px = case["W"] * case["H"] * case["T"]
        spec = _spec(case)
        if kind == "generic":
            return {"bytes": px * ((1 if case["dtype"] == "u8" else 4) + 4), "flops": px * sum(map(_stage_ops, spec))}
        per = (3 if case["chain"] == "rgb_harris" else 1) + (4 if case["chain"] == "grad" else 1)
        return {"bytes": px * per, "flops": px * sum(OPS[o] for o in spec)}
    if kind == "batch":
        px = sum(W * H * T for W, H, T in synth.batch_shapes(case["clip_seed"], case["clips"], case["t_lo"], case["t_hi"]))
        return {"bytes": 2 * px, "flops": px * sum(OPS[o] for o in fz.HARRIS_CHAIN)}
    if kind == "track":
        pts = int((0.93 * case["objects"] + case["clutter"]) * case["T"])
        # the points in, a record a live track and frame out; each track predicted (80 operations), tried
        # against the frame's points (9 each) and updated (60)
        per_frame = pts / case["T"]
        return {"bytes": pts * (16 + 48), "flops": pts * (140 + 9 * per_frame)}
    n, F, h = case["n"], case["features"], 64
    mac = F * h + h * h + h
    P = mac + 2 * h + 1
    if case["predict"]:
        return {"bytes": 4 * (n * (F + 1) + P), "flops": 2 * n * mac}
    return {"bytes": 4 * (n * (F + 1) + 8 * P), "flops": 2 * n * (3 * mac - F * h)}


# ---------------------------------------------------------------- outputs in 64 bits
def _window(x, rx, ry, w=None):
    """Weighted window sum of [T][H][W] with replicated borders (w None: unweighted)."""
    T, H, W = x.shape
    iy = torch.arange(-ry, H + ry, device=x.device).clamp(0, H - 1)
    ix = torch.arange(-rx, W + rx, device=x.device).clamp(0, W - 1)
    p = x[:, iy][:, :, ix]
    out = torch.zeros_like(x)
    for v in range(2 * ry + 1):
        for u in range(2 * rx + 1):
            out.add_(p[:, v:v + H, u:u + W], alpha=1.0 if w is None else float(w[v][u]))
    return out


def _exact_generic(spec, x):
    x = x.to(torch.float64)
    for st in spec:
        if st[0] == "iir":
            a = float(np.float32(st[1]))
            x = x.clone()
            for t in range(1, x.shape[0]):
                x[t] = a * x[t] + (1.0 - a) * x[t - 1]
        elif st[0] == "box":
            x = _window(x, st[1], st[2])
        elif st[0] == "stencil":
            w = np.asarray(st[3], np.float32).astype(np.float64)
            w = w[None] if w.ndim == 2 else w
            T = x.shape[0]
            out = _window(x, st[1], st[2], w[0])
            for tau in range(1, w.shape[0]):
                at = (torch.arange(T, device=x.device) - tau).clamp_min(0)
                out += _window(x[at], st[1], st[2], w[tau])
            x = out
        else:
            k, a, b = st[1], float(np.float32(st[2])), float(np.float32(st[3]))
            x = {"affine": lambda: a * x + b, "abs": x.abs, "square": lambda: x * x, "sqrtabs": lambda: x.abs().sqrt(),
                 "clamp": lambda: x.clamp(a, b)}[k]()
    return x


def _exact_gradient(x):
    x = x.to(torch.float64)
    g = np.exp(-np.arange(-2, 3) ** 2 / 2.0)
    g /= g.sum()
    s = _window(x, 2, 2, np.outer(g, g))
    ix = _window(s, 1, 1, np.outer([1, 2, 1], [-1, 0, 1]))
    iy = _window(s, 1, 1, np.outer([-1, 0, 1], [1, 2, 1]))
    return (ix * ix + iy * iy).sqrt()


def _exact_track(case, seed):
    """Constant-velocity Kalman tracks, greedy nearest neighbour in (distance, id, point) order."""
    pts = _points(case, seed)
    pts = pts[np.lexsort((pts[:, 2], pts[:, 1], pts[:, 0]))].astype(np.float64)
    q, r, gate, v0, max_miss = 0.5, 1.0, 9.21, 4.0, 3
    F = np.eye(4)
    F[0, 2] = F[1, 3] = 1.0
    Q = q * np.array([[.25, 0, .5, 0], [0, .25, 0, .5], [.5, 0, 1, 0], [0, .5, 0, 1]])
    s, P = np.zeros((0, 4)), np.zeros((0, 4, 4))
    ids, miss = np.zeros(0, np.int64), np.zeros(0, np.int64)
    next_id, whole, states = 0, [], []
    bounds = np.searchsorted(pts[:, 0], np.arange(case["T"] + 1))
    for t in range(case["T"]):
        z = pts[bounds[t]:bounds[t + 1]][:, [2, 1]]
        s, P = s @ F.T, F @ P @ F.T + Q
        Si = np.linalg.inv(P[:, :2, :2] + r * np.eye(2)) if len(s) else np.zeros((0, 2, 2))
        nu = z[None] - s[:, None, :2]
        d2 = np.einsum("ija,iab,ijb->ij", nu, Si, nu)
        a, b = np.nonzero(d2 <= gate)
        to, taken = np.full(len(s), -1), np.zeros(len(z), bool)
        for k in np.lexsort((b, ids[a], d2[a, b])):
            if to[a[k]] < 0 and not taken[b[k]]:
                to[a[k]] = b[k]
                taken[b[k]] = True
        hit = to >= 0
        i = np.nonzero(hit)[0]
        K = P[i][:, :, :2] @ Si[i]
        s[i] += np.einsum("iab,ib->ia", K, nu[i, to[i]])
        P[i] -= K @ P[i][:, :2, :]
        miss = np.where(hit, 0, miss + 1)
        live = miss <= max_miss
        fresh = z[~taken]
        k = len(fresh)
        status = np.concatenate([hit[live].astype(np.int64), np.full(k, 2)])
        s = np.concatenate([s[live], np.concatenate([fresh, np.zeros((k, 2))], 1)])
        P = np.concatenate([P[live], np.broadcast_to(np.diag([r, r, v0, v0]), (k, 4, 4))])
        ids = np.concatenate([ids[live], next_id + np.arange(k)])
        miss = np.concatenate([miss[live], np.zeros(k, np.int64)])
        next_id += k
        whole.append(np.stack([np.full(len(ids), t), ids, status], 1))
        states.append(s.copy())
    whole, states = np.concatenate(whole), np.concatenate(states)
    cap = _record_capacity(case)
    rows, cols = np.zeros((cap, 3), np.int32), np.zeros((cap, 4))
    rows[:len(whole)], cols[:len(whole)] = whole, states
    return [np.array([len(whole), 0], np.int32), rows, cols]


def _exact_mlp(case, seed):
    prm, x, t, m, v = (torch.tensor(a.astype(np.float64), device="cuda") for a in _mlp_state(case, seed))
    F, h = case["features"], 64
    prm.requires_grad_(True)
    w1, b1, w2, b2, w3, b3 = prm.split([h * F, h, h * h, h, h, 1])
    y = torch.relu(torch.relu(x @ w1.view(h, F).T + b1) @ w2.view(h, h).T + b2) @ w3 + b3
    if case["predict"]:
        return [y.detach()]
    loss = (y - t).square().mean()
    g, = torch.autograd.grad(loss, prm)
    # the rates as the library is handed them: single precision
    lr, be1, be2, eps = (float(np.float32(c)) for c in (3e-3, 0.9, 0.999, 1e-8))
    m = be1 * m + (1 - be1) * g
    v = be2 * v + (1 - be2) * g * g
    new = prm.detach() - lr * (m / (1 - be1 ** 100)) / ((v / (1 - be2 ** 100)).sqrt() + eps)
    return [loss.detach().reshape(1), g, new, m, v]


def exact(case, seed):
    kind = case["kind"]
    if kind == "track":
        return _exact_track(case, seed)
    if kind == "mlp":
        return _exact_mlp(case, seed)
    if kind == "generic":
        return [_exact_generic(_spec(case), _video(case["W"], case["H"], case["T"], seed))[None]]
    if kind == "chain" and case["chain"] == "grad":
        return [_exact_gradient(_video(case["W"], case["H"], case["T"], seed))[None]]
    return None  # masks and counts: whole numbers

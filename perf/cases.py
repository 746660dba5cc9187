"""Performance cases of the pointmap matcher and of the pose solves that use its matches.

Each case is one pass through the Python entry points of paper_2412_12392_amd
with device inputs that are made from a seed.  The inputs follow the
framework's own synthetic recipe (a pinhole surface seen twice, a random
Sim(3), unit-norm 24-channel descriptors from a smooth field plus noise,
confidences in [1, 5]), drawn on the GPU.

    listed()            the named cases
    draw(rng)           one more case of the same ranges
    prepare(case, seed) the inputs, buffers and parameters of a case
    run(state)          one pass, with its outputs
    work(case)          bytes and operations that one pass cannot do without
    exact(case, seed)   the same outputs from plain torch in 64 bits
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2412_12392_amd as m3s

DEV = "cuda:0"
D = 24

# ---------------------------------------------------------------- the cases


def listed():
    return [
        # Smallest call in use: one low-resolution pair without confidences, where latency counts.
        dict(name="match_64x48", kind="match", W=64, H=48, conf=False, xhat=False, init=False, K=10, r=3, levels=1),
        # The ordinary call: one keyframe pair at the paper's frame size, confidence gate on.
        dict(name="match_512x384", kind="match", W=512, H=384, conf=True, xhat=False, init=False, K=10, r=3, levels=1),
        # A ragged frame whose sides divide no tile, with the sampled point as well.
        dict(name="match_333x247", kind="match", W=333, H=247, conf=True, xhat=True, init=False, K=8, r=2, levels=1),
        # One tracked frame: matching from the previous frame's matches with the coarse-to-fine
        # refine, the keyframe statistics, the pose solve and the fusion into the keyframe.
        dict(name="frame_512x384", kind="frame", W=512, H=384, K=10, r=3, levels=3, iters=10),
        # The pose solve alone on a smaller frame.
        dict(name="track_320x240", kind="track", W=320, H=240, iters=10),
        # Differentiating through one pair: forward with the sampled point, then backward.
        dict(name="train_512x384", kind="train", W=512, H=384, K=10, r=3),
        # The edges of a keyframe graph matched in one call.
        dict(name="batch_64x512x384", kind="batch", W=512, H=384, n=64, mixed=False, K=10, r=3, graph=True),
        # A graph of landscape, portrait and wide frames with their own iteration counts and radii.
        dict(name="batch_mixed_24", kind="batch", W=512, H=384, n=24, mixed=True, K=10, r=3, graph=True),
        # Differentiating through a batch of edges, submitted eagerly.
        dict(name="train_batch_16", kind="train_batch", W=512, H=384, n=16, K=10, r=3),
        # Pose graph of a short sequence of small frames.
        dict(name="backend_8_160x120", kind="backend", W=160, H=120, N=8, loops=1, iters=10),
        # Pose graph of a full-size sequence with three loop closures (65 edges).
        dict(name="backend_32_512x384", kind="backend", W=512, H=384, N=32, loops=3, iters=10),
        # A long sequence of smaller frames with many closures.
        dict(name="backend_96_224x160", kind="backend", W=224, H=160, N=96, loops=8, iters=10),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["match", "match", "frame", "track", "train", "batch", "train_batch", "backend", "backend"])
    W, H = _log(rng, 64, 512), _log(rng, 48, 384)
    if rng.random() < 0.25:
        W, H = H, W
    K, r = rng.randint(5, 15), rng.randint(2, 4)
    if kind == "match":
        return dict(kind=kind, W=W, H=H, conf=rng.random() < 0.7, xhat=rng.random() < 0.4, init=rng.random() < 0.3,
                    K=K, r=r, levels=rng.choice([1, 1, 2, 3]))
    if kind == "frame":
        return dict(kind=kind, W=W, H=H, K=K, r=r, levels=rng.choice([1, 2, 3]), iters=rng.randint(5, 12))
    if kind == "track":
        return dict(kind=kind, W=W, H=H, iters=rng.randint(5, 12))
    if kind == "train":
        return dict(kind=kind, W=W, H=H, K=K, r=r)
    if kind == "batch":
        return dict(kind=kind, W=W, H=H, n=_log(rng, 2, 48), mixed=rng.random() < 0.5, K=min(K, 12), r=min(r, 3),
                    graph=rng.random() < 0.5)
    if kind == "train_batch":
        return dict(kind=kind, W=W, H=H, n=_log(rng, 2, 32), K=min(K, 12), r=min(r, 3))
    N = _log(rng, 5, 100)
    # Long sequences come with smaller frames, so that no drawn graph costs more than the listed one.
    area = min(W * H, 196608 * 30 // N)
    s = math.sqrt(area / (W * H))
    return dict(kind=kind, W=max(40, int(W * s)), H=max(30, int(H * s)), N=N, loops=rng.randint(1, max(1, min(8, N // 4))),
                iters=rng.randint(5, 10))


# ---------------------------------------------------------------- inputs


class _Rng:
    """Seeded draws: small ones on the host, images on the device."""

    def __init__(self, seed):
        self.np = np.random.Generator(np.random.PCG64(seed))
        self.gen = torch.Generator(device=DEV)
        self.gen.manual_seed(seed)

    def normal(self, *shape):
        return torch.randn(*shape, device=DEV, generator=self.gen)

    def uniform(self, lo, hi, *shape):
        return lo + (hi - lo) * torch.rand(*shape, device=DEV, generator=self.gen)


def _sim3(rng, deg, tmax, smin, smax):
    axis = rng.normal(size=3)
    axis /= np.linalg.norm(axis)
    a = math.radians(rng.uniform(0.0, deg))
    k = np.array([[0, -axis[2], axis[1]], [axis[2], 0, -axis[0]], [-axis[1], axis[0], 0]])
    R = np.eye(3) + math.sin(a) * k + (1.0 - math.cos(a)) * (k @ k)
    t = rng.normal(size=3)
    t *= rng.uniform(0.0, tmax) / np.linalg.norm(t)
    return np.concatenate([rng.uniform(smin, smax) * R, t[:, None]], 1)


def _mul(A, B):
    return np.concatenate([A[:, :3] @ B[:, :3], (A[:, :3] @ B[:, 3] + A[:, 3])[:, None]], 1)


def _inv(T):
    s2 = np.cbrt(np.linalg.det(T[:, :3])) ** 2
    Ri = T[:, :3].T / s2
    return np.concatenate([Ri, (-Ri @ T[:, 3])[:, None]], 1)


def _dev(T, dtype=torch.float64):
    return torch.as_tensor(np.asarray(T), dtype=dtype, device=DEV)


def _apply(T, P):
    T = _dev(T)
    return P @ T[:, :3].t() + T[:, 3]


def _grid(H, W):
    y, x = torch.meshgrid(torch.arange(H, device=DEV, dtype=torch.float64),
                          torch.arange(W, device=DEV, dtype=torch.float64), indexing="ij")
    return x, y


def _surface(H, W, x, y):
    f = max(W, H) / 2.0
    u, v = (x - (W - 1) / 2.0) / f, (y - (H - 1) / 2.0) / f
    z = 2.0 + 0.3 * torch.sin(3.0 * u) * torch.cos(2.0 * v) + 0.1 * u + 0.05 * v
    return torch.stack([z * u, z * v, z], -1)


def _field(rng, H, W):
    sig = 2.0 * math.pi * 8.0 / max(W, H)
    om = _dev(rng.np.normal(0.0, sig, size=(8, 2, D)), torch.float32)
    am = _dev(rng.np.normal(0.0, 1.0, size=(8, D)), torch.float32)
    ph = _dev(rng.np.uniform(0.0, 2.0 * math.pi, size=(8, D)), torch.float32)

    def at(x, y):
        x, y = x.float()[..., None], y.float()[..., None]
        out = torch.zeros((*x.shape[:-1], D), device=DEV)
        for k in range(8):
            out += am[k] * torch.sin(om[k, 0] * x + om[k, 1] * y + ph[k])
        out += 0.05 * rng.normal(*out.shape)
        return (out / out.norm(dim=-1, keepdim=True)).contiguous()

    return at


def _pair(rng, H, W, conf=True, init=False, small_motion=False):
    """One matching problem: reference and query pointmaps, descriptors, confidences, initial pixels."""
    x, y = _grid(H, W)
    Xii = _surface(H, W, x, y).float()
    d = rng.np.uniform(-2.0, 2.0, size=2)
    T = _sim3(rng.np, 4.0, 0.05, 0.97, 1.03) if small_motion else _sim3(rng.np, 10.0, 0.1, 0.9, 1.1)
    Xji = (_apply(T, _surface(H, W, x + d[0], y + d[1])) + 1e-3 * rng.normal(H, W, 3)).float()
    P, f = Xji.double(), max(W, H) / 2.0
    px, py = f * P[..., 0] / P[..., 2] + (W - 1) / 2.0, f * P[..., 1] / P[..., 2] + (H - 1) / 2.0
    at = _field(rng, H, W)
    p = dict(Xii=Xii.contiguous(), Xji=Xji.contiguous(), Dii=at(x, y), Dji=at(px, py), Qii=None, Qji=None, p_init=None)
    if conf:
        p["Qii"], p["Qji"] = rng.uniform(1.0, 5.0, H, W), rng.uniform(1.0, 5.0, H, W)
    if init:
        p["p_init"] = (torch.stack([px, py], -1).float() + 1.5 * rng.normal(H, W, 2)).contiguous()
    return p


def _args(p):
    return (p["Xii"], p["Xji"], p["Dii"], p["Dji"], p["Qii"], p["Qji"], p["p_init"])


def _grads(rng, H, W):
    """Gradients that a loss sends back into p* and the sampled point."""
    return 0.1 * rng.normal(H, W, 2), rng.normal(H, W, 3)


def _batch_spec(case):
    """(H, W, K, r) of every edge of a batch."""
    n, H, W = case["n"], case["H"], case["W"]
    if not case.get("mixed"):
        return [(H, W, case["K"], case["r"])] * n
    rng = np.random.Generator(np.random.PCG64(4000 + n))
    shapes = [(H, W), (W, H), (max(8, 3 * H // 4), W)]
    return [(*shapes[int(rng.choice(3, p=[0.42, 0.33, 0.25]))], int(rng.integers(max(1, case["K"] - 5), case["K"] + 6)),
             int(rng.integers(max(1, case["r"] - 1), case["r"] + 2))) for _ in range(n)]


def _flat_outputs(spec, xhat):
    """Output buffers of a batch, one allocation per kind, and each edge's views of them."""
    total = sum(H * W for H, W, _, _ in spec)
    flat = dict(p=torch.empty(2 * total, device=DEV), idx=torch.empty(total, dtype=torch.int32, device=DEV),
                valid=torch.empty(total, dtype=torch.uint8, device=DEV), theta=torch.empty(total, device=DEV))
    if xhat:
        flat["xhat"] = torch.empty(3 * total, device=DEV)
    outs, o = [], 0
    for H, W, _, _ in spec:
        n = H * W
        outs.append(m3s.MatchResult(flat["p"][2 * o:2 * (o + n)].view(H, W, 2), flat["idx"][o:o + n].view(H, W),
                                    flat["valid"][o:o + n].view(H, W), flat["theta"][o:o + n].view(H, W),
                                    flat["xhat"][3 * o:3 * (o + n)].view(H, W, 3) if xhat else None))
        o += n
    return flat, outs


def _backend_inputs(case, rng):
    """Keyframes that pan over one surface: matches are shifted pixels, both ways between
    neighbours, plus loop closures; initial poses off by a small Sim(3)."""
    N, H, W = case["N"], case["H"], case["W"]
    x, y = _grid(H, W)
    T_true, T_init, shift = [], [], []
    step = max(1, min(H, W) // 20)
    for k in range(N):
        T = np.eye(3, 4) if k == 0 else _mul(T_true[-1], _sim3(rng.np, 4.0, 0.1, 0.97, 1.03))
        T_true.append(T)
        T_init.append(T if k == 0 else _mul(_sim3(rng.np, 2.0, 0.02, 0.98, 1.02), T))
        # The pan reflects at a third of the frame, so that loop closures overlap too.
        s = np.zeros(2, int) if k == 0 else shift[-1] + rng.np.integers(-step, step + 1, size=2)
        shift.append(np.clip(s, [-W // 6, -H // 6], [W // 6, H // 6]))
    Xc = torch.empty(N, H, W, 3, device=DEV)
    for k in range(N):
        P = _surface(H, W, x + float(shift[k][0]), y + float(shift[k][1]))
        Xc[k] = (_apply(_inv(T_true[k]), P) + 2e-3 * rng.normal(H, W, 3)).float()
    pairs = [e for k in range(1, N) for e in ((k - 1, k), (k, k - 1))]
    pairs += [(c, N - 1 - c) for c in range(case["loops"]) if N - 1 - 2 * c > 1]
    E = len(pairs)
    idx = torch.empty(E, H, W, dtype=torch.int32, device=DEV)
    valid = torch.empty(E, H, W, dtype=torch.uint8, device=DEV)
    for e, (i, j) in enumerate(pairs):
        d = shift[j] - shift[i]
        mx, my = x + float(d[0]), y + float(d[1])
        inside = (mx >= 0) & (mx < W) & (my >= 0) & (my < H)
        idx[e] = torch.where(inside, my * W + mx, torch.full_like(mx, -1.0)).int()
        valid[e] = (inside & (rng.uniform(0.0, 1.0, H, W) < 0.95)).to(torch.uint8)
    return dict(Xc=Xc, Q=rng.uniform(1.0, 5.0, N, H, W), edges=_dev(pairs, torch.int32), idx=idx, valid=valid,
                T0=_dev(np.stack(T_init), torch.float32))


def prepare(case, seed):
    rng = _Rng(seed)
    kind, H, W = case["kind"], case["H"], case["W"]
    s = dict(kind=kind, case=case)
    if kind == "match":
        s["pair"] = _pair(rng, H, W, case["conf"], case["init"])
        s["prm"] = m3s.params(max_iter=case["K"], refine_radius=case["r"], refine_levels=case["levels"])
    elif kind == "frame":
        # The keyframe's pixels are the queries and the frame is the reference.
        s["pair"] = _pair(rng, H, W, True, True, small_motion=True)
        s["prm"] = m3s.params(max_iter=case["K"], refine_radius=case["r"], refine_levels=case["levels"])
        s["tprm"] = m3s.track_params(iters=case["iters"])
        # The keyframe's own points (what the pose maps the frame's points onto).
        T = _sim3(rng.np, 2.0, 0.03, 0.98, 1.02)
        s["Xk"] = _apply(T, s["pair"]["Xji"].double()).float().contiguous()
        s["T0"] = _dev(_mul(_sim3(rng.np, 0.5, 0.01, 0.995, 1.005), T), torch.float32).contiguous()
        s["Xc"], s["Cc"] = s["Xk"].clone(), rng.uniform(0.5, 20.0, H, W)
        s["C"] = rng.uniform(1.0, 5.0, H, W)
    elif kind == "track":
        s.update(_track_inputs(rng, H, W))
        s["tprm"] = m3s.track_params(iters=case["iters"])
    elif kind == "train":
        s["pair"] = _pair(rng, H, W)
        s["pair"]["Xii"].requires_grad_(True)
        s["pair"]["Xji"].requires_grad_(True)
        s["prm"] = m3s.params(max_iter=case["K"], refine_radius=case["r"])
        s["gp"], s["gx"] = _grads(rng, H, W)
    elif kind in ("batch", "train_batch"):
        spec = _batch_spec(case)
        xhat = kind == "train_batch"
        s["pairs"] = [_pair(rng, h, w) for h, w, _, _ in spec]
        s["prm"] = m3s.params(max_iter=case["K"], refine_radius=case["r"])
        s["edges"] = [m3s.EdgeInput(*_args(p), max_iter=k, refine_radius=r) for p, (_, _, k, r) in zip(s["pairs"], spec)]
        s["flat"], s["outs"] = _flat_outputs(spec, xhat)
        if xhat:
            n = case["n"]
            s["dXii"], s["dXji"] = torch.empty(n, H, W, 3, device=DEV), torch.empty(n, H, W, 3, device=DEV)
            s["g"] = [_grads(rng, H, W) for _ in range(n)]
            s["bwd"] = [m3s.BwdEdgeInput(p["Xii"], p["Xji"], o.p, o.valid, gp, gx)
                        for p, o, (gp, gx) in zip(s["pairs"], s["outs"], s["g"])]
            s["gouts"] = [(s["dXii"][k], s["dXji"][k]) for k in range(n)]
    elif kind == "backend":
        s.update(_backend_inputs(case, rng))
        s["bprm"] = m3s.backend_params(iters=case["iters"])
    return s


def _track_inputs(rng, H, W):
    x, y = _grid(H, W)
    Xf = _surface(H, W, x, y)
    T = _sim3(rng.np, 5.0, 0.05, 0.95, 1.05)
    dx, dy = (int(v) for v in rng.np.integers(-6, 7, size=2))
    mx, my = (x + dx).clamp(0, W - 1).long(), (y + dy).clamp(0, H - 1).long()
    idx = my * W + mx
    Xk = _apply(T, Xf.view(-1, 3)[idx.view(-1)]).view(H, W, 3) + 1e-3 * rng.normal(H, W, 3)
    bad = rng.uniform(0.0, 1.0, H, W) < 0.05
    Xk = Xk + bad[..., None] * 0.5 * rng.normal(H, W, 3)
    return dict(Xk=Xk.float().contiguous(), Xf=Xf.float().contiguous(), idx=idx.int(),
                valid=(rng.uniform(0.0, 1.0, H, W) < 0.95).to(torch.uint8), Qf=rng.uniform(1.0, 5.0, H, W),
                Qk=rng.uniform(1.0, 5.0, H, W), T0=_dev(np.eye(3, 4), torch.float32))


# ---------------------------------------------------------------- one pass


def run(s):
    kind = s["kind"]
    if kind == "match":
        return _named(m3s.match(*_args(s["pair"]), s["prm"], want_xhat=s["case"]["xhat"]))
    if kind == "frame":
        p = s["pair"]
        res = m3s.match(*_args(p), s["prm"])
        counts = m3s.match_stats(res)
        T, info = m3s.track_pose(s["Xk"], p["Xii"], res.idx, res.valid, p["Qii"], p["Qji"], s["T0"].clone(), s["tprm"])
        Xc, Cc = m3s.fuse_pointmap(s["Xc"], s["Cc"], p["Xji"], s["C"], T)
        return dict(_named(res), counts=counts, T=T, info=info, Xc=Xc, Cc=Cc)
    if kind == "track":
        T, info = m3s.track_pose(s["Xk"], s["Xf"], s["idx"], s["valid"], s["Qf"], s["Qk"], s["T0"].clone(), s["tprm"])
        return dict(T=T, info=info)
    if kind == "train":
        p = s["pair"]
        pm, xhat, idx, valid, theta = m3s.MatchFunction.apply(*_args(p), s["prm"])
        gi, gj = torch.autograd.grad((pm, xhat), (p["Xii"], p["Xji"]), (s["gp"], s["gx"]))
        return dict(p=pm, xhat=xhat, idx=idx, valid=valid, theta=theta, dXii=gi, dXji=gj)
    if kind == "batch":
        m3s.match_batched(s["edges"], s["prm"], graph=s["case"]["graph"], outs=s["outs"])
        return s["flat"]
    if kind == "train_batch":
        m3s.match_batched(s["edges"], s["prm"], graph=False, outs=s["outs"])
        m3s.match_backward_batched(s["bwd"], graph=False, outs=s["gouts"])
        return dict(s["flat"], dXii=s["dXii"], dXji=s["dXji"])
    T, info = m3s.backend_gn(s["Xc"], s["Q"], s["edges"], s["idx"], s["valid"], s["T0"].clone(), s["bprm"])
    return dict(T=T, info=info)


def _named(res):
    d = dict(p=res.p, idx=res.idx, valid=res.valid, theta=res.theta)
    if res.xhat is not None:
        d["xhat"] = res.xhat
    return d


# ---------------------------------------------------------------- work


def _match_work(n, K, r, levels=1, conf=True, init=False, xhat=False):
    # Points 12 + 12, descriptors 96 + 96, p 8, idx 4, valid 1, theta 4 per pixel.
    b = n * (24 + 192 + 17 + (8 if conf else 0) + (8 if init else 0) + (12 if xhat else 0))
    # About 110 operations per ray sample and step, 2 D per scored candidate.
    return b, n * (110.0 * (K + 1) + 2.0 * D * levels * (2 * r + 1) ** 2)


def work(case):
    kind, n = case["kind"], case["H"] * case["W"]
    if kind == "match":
        b, f = _match_work(n, case["K"], case["r"], case["levels"], case["conf"], case["init"], case["xhat"])
    elif kind == "frame":
        b, f = _match_work(n, case["K"], case["r"], case["levels"], True, True)
        # The keyframe's points once more, the canonical map and confidence in and out, the frame's confidence.
        b, f = b + n * (12 + 16 + 16 + 4), f + n * 100.0 * (case["iters"] + 1)
    elif kind == "track":
        b, f = n * 37, n * 100.0 * (case["iters"] + 1)
    elif kind == "train":
        b, f = _match_work(n, case["K"], case["r"], xhat=True)
        b, f = b + n * (20 + 24), f + n * 300.0
    elif kind in ("batch", "train_batch"):
        b = f = 0
        for H, W, K, r in _batch_spec(case):
            x, y = _match_work(H * W, K, r, xhat=kind == "train_batch")
            b, f = b + x, f + y
        if kind == "train_batch":
            b, f = b + case["n"] * n * (20 + 24), f + case["n"] * n * 300.0
    else:
        N = case["N"]
        E = 2 * (N - 1) + sum(1 for c in range(case["loops"]) if N - 1 - 2 * c > 1)
        b, f = n * (16 * N + 5 * E), 100.0 * n * E * (case["iters"] + 1)
    return dict(bytes=b, flops=f)


# ---------------------------------------------------------------- 64-bit results


def _rays(X):
    X = X.double()
    n2 = (X * X).sum(-1, keepdim=True)
    ok = torch.isfinite(X).all(-1, keepdim=True) & (n2 > 0) & torch.isfinite(n2)
    return torch.where(ok, X / n2.clamp_min(1e-300).sqrt(), torch.zeros_like(X))


def _ray_image(X):
    """Unit rays and their central-difference gradients, 9 channels per pixel."""
    R = _rays(X)
    H, W = R.shape[:2]
    xs, ys = torch.arange(W, device=R.device), torch.arange(H, device=R.device)
    xm, xp, ym, yp = (xs - 1).clamp_min(0), (xs + 1).clamp_max(W - 1), (ys - 1).clamp_min(0), (ys + 1).clamp_max(H - 1)
    gx = (R[:, xp] - R[:, xm]) / (xp - xm).double()[None, :, None]
    gy = (R[yp] - R[ym]) / (yp - ym).double()[:, None, None]
    return torch.cat([R, gx, gy], -1).view(H * W, 9)


def _cell(p, H, W):
    x0 = p[:, 0].floor().clamp_max(W - 2)
    y0 = p[:, 1].floor().clamp_max(H - 2)
    a, b = p[:, 0] - x0, p[:, 1] - y0
    m = (y0 * W + x0).long()
    corners = torch.stack([m, m + 1, m + W, m + W + 1], 1)
    w = torch.stack([(1 - a) * (1 - b), a * (1 - b), (1 - a) * b, a * b], 1)
    return corners, w, a, b


def _sample(img, p, H, W, t):
    corners, w, _, _ = _cell(p, H, W)
    s = (img[corners] * w[..., None]).sum(1)
    r = s[:, :3]
    n = r.norm(dim=1, keepdim=True)
    psi = r / n
    e = psi - t
    jx = (s[:, 3:6] - psi * (psi * s[:, 3:6]).sum(1, keepdim=True)) / n
    jy = (s[:, 6:9] - psi * (psi * s[:, 6:9]).sum(1, keepdim=True)) / n
    c = (e * e).sum(1)
    c = torch.where(torch.isfinite(c) & (n[:, 0] > 0), c, torch.full_like(c, math.inf))
    return c, (jx * jx).sum(1), (jx * jy).sum(1), (jy * jy).sum(1), (jx * e).sum(1), (jy * e).sum(1)


def _exact_match(p, K, r, levels, prm, xhat, want_idx):
    H, W = p["Xii"].shape[:2]
    n = H * W
    img, t = _ray_image(p["Xii"]), _rays(p["Xji"]).view(n, 3)
    hi = torch.tensor([W - 1.0, H - 1.0], dtype=torch.float64, device=DEV)
    if p["p_init"] is not None:
        q = p["p_init"].double().view(n, 2)
    else:
        x, y = _grid(H, W)
        q = torch.stack([x, y], -1).view(n, 2)
    q = torch.minimum(q.clamp_min(0.0), hi)
    lam = torch.full((n,), float(prm.lambda_init), dtype=torch.float64, device=DEV)
    cur = _sample(img, q, H, W, t)
    for _ in range(K):
        c, a00, a01, a11, g0, g1 = cur
        b00, b11 = a00 + lam, a11 + lam
        det = b00 * b11 - a01 * a01
        d = torch.stack([-(b11 * g0 - a01 * g1) / det, -(b00 * g1 - a01 * g0) / det], 1)
        fine = torch.isfinite(d).all(1)
        hold = ((q <= 0) & (d < 0)) | ((q >= hi) & (d > 0))
        alone = torch.stack([-g0 / b00, -g1 / b11], 1)
        d = torch.where(hold.any(1, keepdim=True), torch.where(hold, torch.zeros_like(d), alone), d)
        trial = torch.minimum((q + torch.where(fine[:, None], d, torch.zeros_like(d))).clamp_min(0.0), hi)
        nxt = _sample(img, trial, H, W, t)
        acc = fine & (nxt[0] < c)
        q = torch.where(acc[:, None], trial, q)
        cur = tuple(torch.where(acc, u, v) for u, v in zip(nxt, cur))
        lam = torch.where(acc, lam * 0.1, lam * 10.0)
    theta = 2.0 * torch.asin((cur[0].sqrt() * 0.5).clamp_max(1.0))
    out = dict(p=q.view(H, W, 2), idx=None, valid=None, theta=theta.view(H, W))
    if xhat:
        corners, w, _, _ = _cell(q, H, W)
        out["xhat"] = (p["Xii"].double().view(n, 3)[corners] * w[..., None]).sum(1).view(H, W, 3)
    if want_idx:
        Di, Dj = p["Dii"].double().view(n, D), p["Dji"].double().view(n, D)
        cx, cy = (q[:, 0] + 0.5).floor().long(), (q[:, 1] + 0.5).floor().long()
        for lev in reversed(range(levels)):
            best = torch.full((n,), -math.inf, dtype=torch.float64, device=DEV)
            bm = torch.zeros(n, dtype=torch.long, device=DEV)
            for dy in range(-r, r + 1):
                for dx in range(-r, r + 1):
                    mx, my = cx + (dx << lev), cy + (dy << lev)
                    inside = (mx >= 0) & (mx < W) & (my >= 0) & (my < H)
                    m = torch.where(inside, my * W + mx, torch.zeros_like(mx))
                    sc = torch.where(inside, (Di[m] * Dj).sum(1), torch.full_like(best, -math.inf))
                    up = sc > best
                    best, bm = torch.where(up, sc, best), torch.where(up, m, bm)
            cx, cy = bm % W, bm // W
        ok = theta <= prm.max_theta
        if p["Qii"] is not None:
            ok &= (p["Qii"].double().view(n)[bm] * p["Qji"].double().view(n)).sqrt() >= prm.conf_min
        out["idx"], out["valid"] = bm, ok
    return out


def _proj(X, v):
    n = X.norm(dim=-1, keepdim=True)
    u = X / n
    return (v - u * (u * v).sum(-1, keepdim=True)) / n


def _exact_backward(Xii, Xji, q, ok, gp, gx):
    H, W = Xii.shape[:2]
    n = H * W
    X, x = Xii.double().view(n, 3), Xji.double().view(n, 3)
    R = _rays(Xii).view(n, 3)
    hi = torch.tensor([W - 1.0, H - 1.0], dtype=torch.float64, device=DEV)
    q, gp, gx = q.view(n, 2), gp.double().view(n, 2), gx.double().view(n, 3)
    corners, w, a, b = _cell(q, H, W)
    a, b = a[:, None], b[:, None]

    def slopes(v):
        return ((1 - b) * (v[:, 1] - v[:, 0]) + b * (v[:, 3] - v[:, 2]), (1 - a) * (v[:, 2] - v[:, 0]) + a * (v[:, 3] - v[:, 1]))

    Rc, Xcn = R[corners], X[corners]
    rs = (Rc * w[..., None]).sum(1)
    j0, j1 = (_proj(rs, d) for d in slopes(Rc))
    dx0, dx1 = slopes(Xcn)
    g0, g1 = gp[:, 0] + (dx0 * gx).sum(1), gp[:, 1] + (dx1 * gx).sum(1)
    a00, a01, a11 = (j0 * j0).sum(1), (j0 * j1).sum(1), (j1 * j1).sum(1)
    held = (q <= 0) | (q >= hi)
    det = a00 * a11 - a01 * a01
    m0, m1 = (a11 * g0 - a01 * g1) / det, (a00 * g1 - a01 * g0) / det
    m0 = torch.where(held[:, 0], torch.zeros_like(m0), torch.where(held[:, 1], g0 / a00, m0))
    m1 = torch.where(held[:, 1], torch.zeros_like(m1), torch.where(held[:, 0], g1 / a11, m1))
    v = j0 * m0[:, None] + j1 * m1[:, None]
    okd = ok.double()[:, None]
    dXji = _proj(x, v) * okd
    dXii = torch.zeros_like(X)
    for c in range(4):
        wc = w[:, c:c + 1]
        dXii.index_add_(0, corners[:, c], (wc * gx - wc / rs.norm(dim=1, keepdim=True) * _proj(Xcn[:, c], v)) * okd)
    return dXii.view(H, W, 3), dXji.view(H, W, 3)


def _normal(T, X, Y, q, prm):
    """Normal equations, robust cost and count of matches x = T X against Y (a left perturbation of T)."""
    x = X @ T[:, :3].t() + T[:, 3]
    d, dy = x.norm(dim=1, keepdim=True), Y.norm(dim=1, keepdim=True)
    ok = (d > 0) & (dy > 0) & (q[:, None] > prm.q_min)
    x, Y, q, d, dy = (v[ok[:, 0]] for v in (x, Y, q, d, dy))
    u = x / d
    e, rd = u - Y / dy, (d - dy)[:, 0]
    Z, I = torch.zeros_like(d[:, 0]), torch.eye(3, dtype=torch.float64, device=DEV)
    P = I - u[:, :, None] * u[:, None, :]
    S = torch.stack([Z, -x[:, 2], x[:, 1], x[:, 2], Z, -x[:, 0], -x[:, 1], x[:, 0], Z], 1).view(-1, 3, 3)
    Jr = torch.cat([P / d[..., None], -S / d[..., None], torch.zeros_like(S[:, :, :1])], 2)
    Jd = torch.cat([u, torch.zeros_like(u), d], 1)
    ar, ad = e.norm(dim=1) * q.sqrt() / prm.sigma_ray, rd.abs() * q.sqrt() / prm.sigma_dist
    k = prm.huber

    def rob(v):
        far = v > k
        return torch.where(far, k / v.clamp_min(1e-300), torch.ones_like(v)), torch.where(far, k * (v - 0.5 * k), 0.5 * v * v)

    (hr, cr), (hd, cd) = rob(ar), rob(ad)
    J = torch.cat([Jr * (q / prm.sigma_ray ** 2 * hr).sqrt()[:, None, None], (Jd * (q / prm.sigma_dist ** 2 * hd).sqrt()[:, None])[:, None]], 1)
    res = torch.cat([e * (q / prm.sigma_ray ** 2 * hr).sqrt()[:, None], (rd * (q / prm.sigma_dist ** 2 * hd).sqrt())[:, None]], 1)
    J, res = J.reshape(-1, 7), res.reshape(-1)
    return J.t() @ J, J.t() @ res, float((cr + cd).sum()), q.numel()


def _exp(tau):
    v, w, s = tau[:3], tau[3:6], float(tau[6])
    G = torch.zeros(4, 4, dtype=torch.float64)
    G[0, 1], G[0, 2], G[1, 0], G[1, 2], G[2, 0], G[2, 1] = -w[2], w[1], w[2], -w[0], -w[1], w[0]
    G[:3, :3] += s * torch.eye(3, dtype=torch.float64)
    G[:3, 3] = v
    return torch.linalg.matrix_exp(G)[:3].numpy()


def _exact_track(Xk, Xf, idx, valid, Qf, Qk, T0, prm):
    ok = valid.reshape(-1).bool() & (idx.reshape(-1) >= 0)
    m = idx.reshape(-1).long()[ok]
    X, Y = Xf.double().view(-1, 3)[m], Xk.double().view(-1, 3)[ok]
    q = (Qf.double().view(-1)[m] * Qk.double().view(-1)[ok]).sqrt()
    T, last = T0.double().cpu().numpy(), 0.0
    for _ in range(prm.iters):
        Hm, g, _, _ = _normal(_dev(T), X, Y, q, prm)
        tau = torch.linalg.solve(Hm.cpu(), -g.cpu())
        T, last = _mul(_exp(tau), T), float(tau.norm())
    _, _, cost, count = _normal(_dev(T), X, Y, q, prm)
    return _dev(T), torch.tensor([cost, float(count), float(prm.iters), last], dtype=torch.float64)


def _adjoint(T):
    s = np.cbrt(np.linalg.det(T[:, :3]))
    R, t = T[:, :3] / s, T[:, 3]
    A = np.zeros((7, 7))
    A[:3, :3], A[3:6, 3:6], A[:3, 6], A[6, 6] = s * R, R, -t, 1.0
    A[:3, 3:6] = np.array([[0, -t[2], t[1]], [t[2], 0, -t[0]], [-t[1], t[0], 0]]) @ R
    return A


def _exact_backend(s):
    N = s["Xc"].shape[0]
    Xc, Q = s["Xc"].view(N, -1, 3), s["Q"].view(N, -1)
    T = [t.double().cpu().numpy() for t in s["T0"]]
    edges, prm = s["edges"].cpu().numpy(), s["bprm"]
    oks = [(s["valid"][e].view(-1).bool() & (s["idx"][e].view(-1) >= 0)) for e in range(len(edges))]

    def system(e):
        i, j = edges[e]
        m = s["idx"][e].view(-1).long()[oks[e]]
        q = (Q[i].double()[m] * Q[j].double()[oks[e]]).sqrt()
        return _normal(_dev(_mul(_inv(T[i]), T[j])), Xc[j].double()[oks[e]], Xc[i].double()[m], q, prm)

    last = 0.0
    for _ in range(prm.iters):
        Hm, g = np.zeros((N, N, 7, 7)), np.zeros((N, 7))
        for e, (i, j) in enumerate(edges):
            h, b, _, _ = system(e)
            A = _adjoint(_inv(T[i]))
            h, b = A.T @ h.cpu().numpy() @ A, A.T @ b.cpu().numpy()
            Hm[i, i] += h
            Hm[j, j] += h
            Hm[i, j] -= h
            Hm[j, i] -= h.T
            g[i] -= b
            g[j] += b
        full = Hm[1:, 1:].transpose(0, 2, 1, 3).reshape(7 * (N - 1), -1)
        tau = np.linalg.solve(full, -g[1:].reshape(-1))
        last = float(np.linalg.norm(tau))
        for k in range(1, N):
            T[k] = _mul(_exp(torch.from_numpy(tau[7 * (k - 1):7 * k])), T[k])
    cost, count = 0.0, 0.0
    for e in range(len(edges)):
        _, _, c, k = system(e)
        cost, count = cost + c, count + k
    return dict(T=_dev(np.stack(T)), info=torch.tensor([cost, count, float(prm.iters), last], dtype=torch.float64))


def exact(case, seed):
    s = prepare(case, seed)
    kind, H, W = case["kind"], case["H"], case["W"]
    if kind == "match":
        return _exact_match(s["pair"], case["K"], case["r"], case["levels"], s["prm"], case["xhat"], False)
    if kind == "frame":
        p = s["pair"]
        o = _exact_match(p, case["K"], case["r"], case["levels"], s["prm"], False, True)
        T, _ = _exact_track(s["Xk"], p["Xii"], o["idx"], o["valid"], p["Qii"], p["Qji"], s["T0"], s["tprm"])
        Cc, C = s["Cc"].double(), s["C"].double()
        Xc = (Cc[..., None] * s["Xc"].double() + C[..., None] * _apply(T.cpu().numpy(), p["Xji"].double())) / (Cc + C)[..., None]
        return dict(o, idx=None, valid=None, counts=None, T=T, info=None, Xc=Xc, Cc=Cc + C)
    if kind == "track":
        T, info = _exact_track(s["Xk"], s["Xf"], s["idx"], s["valid"], s["Qf"], s["Qk"], s["T0"], s["tprm"])
        return dict(T=T, info=info)
    if kind == "train":
        p = {k: None if v is None else v.detach() for k, v in s["pair"].items()}
        o = _exact_match(p, case["K"], case["r"], 1, s["prm"], True, True)
        gi, gj = _exact_backward(p["Xii"], p["Xji"], o["p"], o["valid"], s["gp"], s["gx"])
        return dict(o, idx=None, valid=None, dXii=gi, dXji=gj)
    if kind in ("batch", "train_batch"):
        grad = kind == "train_batch"
        got = [_exact_match(p, k, r, 1, s["prm"], grad, grad) for p, (_, _, k, r) in zip(s["pairs"], _batch_spec(case))]
        out = {k: torch.cat([o[k].reshape(-1) for o in got]) for k in (("p", "theta", "xhat") if grad else ("p", "theta"))}
        out.update(idx=None, valid=None)
        if grad:
            d = [_exact_backward(p["Xii"], p["Xji"], o["p"], o["valid"], gp, gx)
                 for p, o, (gp, gx) in zip(s["pairs"], got, s["g"])]
            out["dXii"], out["dXji"] = torch.stack([x for x, _ in d]), torch.stack([x for _, x in d])
        return out
    return _exact_backend(s)

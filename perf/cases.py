"""Timed workloads of pprs: what programs built on the package call, over the sizes they use.

listed() names the standing cases and draw() gives further ones of the same ranges. prepare()
makes the inputs of a case on the GPU from a seed, run() takes one pass through the package's
public entry points, work() counts what a pass cannot do without, and exact() is the same result
in FP64 from plain torch.

Inputs are micrograph-like frames: a square lattice of Gaussian blobs seen through a per-frame
drift and a smooth warp, with Poisson counting noise (the statistics of the synthetic series the
benchmark registers), or what such frames become on the way to the network.
"""
import json
import math
import os

import numpy as np
import torch
import torch.nn.functional as F

import paper_1712_02533_amd as P

WEIGHTS = os.path.join(os.path.dirname(os.path.abspath(P.__file__)), "weights",
                       "warmstart_512.safetensors")
DEVICE = "cuda:0"


# ---- the cases --------------------------------------------------------------------------------

def levels_of(side):
    """Grid levels of a frame side: the coarsest level is 6 (65 nodes), 5 for the smallest."""
    return max(2, side.bit_length() - 1 - 5)


def listed():
    return [
        # one interactive registration of two small frames: latency and launches count
        {"name": "pair_64", "kind": "pair", "side": 64, "levels": 2, "init": False, "counts": 20.0},
        # one full-size registration from a composed guess, as each scan operator application is
        {"name": "pair_512_init", "kind": "pair", "side": 512, "levels": 4, "init": True,
         "counts": 5.0},
        # a handful of frame pairs checked together before a series is run (odd node-grid frames)
        {"name": "pairs_16x257", "kind": "pairs", "pairs": 16, "side": 257, "levels": 3,
         "counts": 10.0},
        # an ordinary short series
        {"name": "series_64x256", "kind": "series", "frames": 64, "side": 256, "levels": 3,
         "scan": "brent_kung", "start": "cold", "counts": 10.0},
        # the benchmark series: the largest call
        {"name": "series_512x512", "kind": "series", "frames": 512, "side": 512, "levels": 4,
         "scan": "brent_kung", "start": "cold", "counts": 5.0},
        # a series whose registrations start from the learned warm start
        {"name": "warm_97x512", "kind": "series", "frames": 97, "side": 512, "levels": 4,
         "scan": "brent_kung", "start": "skip", "counts": 5.0},
        # uneven series of one session sharing a pool
        {"name": "batch_mixed", "kind": "batch", "sides": "128,256,512,1024,128,256",
         "lengths": "45,33,24,9,70,17", "counts": 8.0},
        # drift correction alone: the rigid operator over a series of large frames
        {"name": "rigid_96x1024", "kind": "rigid", "frames": 96, "side": 1024, "levels": 3,
         "scan": "brent_kung", "counts": 10.0},
        # one round of the averaging procedure on an aligned series
        {"name": "refine_24x256", "kind": "refine", "frames": 24, "side": 256, "levels": 3,
         "counts": 10.0},
        # the averaged image of an aligned full-size series
        {"name": "average_512x512", "kind": "average", "frames": 512, "height": 512,
         "width": 512},
        # the warm-start network: predictions for the neighbour pairs of a 512-frame series
        {"name": "net_forward_511", "kind": "forward", "batch": 511},
        # the warm-start network: loss and parameter gradients of one training batch
        {"name": "net_gradients_64", "kind": "gradients", "batch": 64},
    ]


def log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["pair", "pair", "pairs", "series", "series", "series", "batch", "rigid",
                       "refine", "average", "forward", "gradients"])
    counts = round(rng.uniform(2.0, 20.0), 2)
    side = rng.choice([64, 128, 256, 512]) + rng.choice([0, 0, 1])  # pixels or grid nodes
    px = side * side
    if kind == "pair":
        side = rng.choice([64, 65, 128, 256, 257, 512, 513, 1024])
        return {"kind": kind, "side": side, "levels": levels_of(side),
                "init": rng.random() < 0.5, "counts": counts}
    if kind == "pairs":
        return {"kind": kind, "pairs": log_int(rng, 1, min(200, (64 << 18) // px)), "side": side,
                "levels": levels_of(side), "counts": counts}
    if kind == "series":
        scan = rng.choice(["brent_kung", "brent_kung", "brent_kung", "general", "blelloch",
                           "sklansky", "sequential"])
        most = min(512, (128 << 18) // px) // (16 if scan == "sequential" else 1)
        start = rng.choice(["cold", "cold", "skip", "refine"]) if side >= 128 else "cold"
        return {"kind": kind, "frames": log_int(rng, 3, most), "side": side,
                "levels": levels_of(side), "scan": scan, "start": start, "counts": counts}
    if kind == "batch":
        sides = [rng.choice([64, 128, 256, 512]) for _ in range(rng.randint(2, 8))]
        return {"kind": kind, "sides": ",".join(map(str, sides)),
                "lengths": ",".join(str(log_int(rng, 2, min(96, (24 << 18) // (s * s))))
                                    for s in sides), "counts": counts}
    if kind == "rigid":
        side = rng.choice([128, 256, 512, 1024])
        return {"kind": kind, "frames": log_int(rng, 2, min(300, (256 << 18) // (side * side))),
                "side": side, "levels": levels_of(side),
                "scan": rng.choice(["brent_kung", "general"]), "counts": counts}
    if kind == "refine":
        return {"kind": kind, "frames": log_int(rng, 3, min(96, (48 << 18) // px)), "side": side,
                "levels": levels_of(side), "counts": counts}
    if kind == "average":
        h, w = log_int(rng, 50, 1100), log_int(rng, 50, 1100)
        return {"kind": kind, "frames": log_int(rng, 2, min(1000, (512 << 18) // (h * w))),
                "height": h, "width": w}
    return {"kind": kind, "batch": log_int(rng, 1, 511 if kind == "forward" else 64)}


# ---- inputs -----------------------------------------------------------------------------------

def blob_frames(seed, n, height, width, drift, warp, counts):
    """[n, height, width] float32 on the GPU and the frames' drifts [n, 2] (x, y) in pixels.
    Lattice spacing 6 px, blob sigma 1.5 px, amplitudes U[0.5, 1]; per frame a drift U[-D, D]^2
    and four sinusoids of amplitude U[0, A/4], wavelength U[32, 128] px; Poisson counts."""
    rng = np.random.default_rng([seed, 11])
    spacing, sigma = 6.0, 1.5
    pad = int(math.ceil((drift + warp) / spacing)) + 4
    ny, nx = int(height / spacing) + 2 * pad + 2, int(width / spacing) + 2 * pad + 2
    amps = torch.tensor(rng.uniform(0.5, 1.0, ny * nx), device=DEVICE, dtype=torch.float32)
    origin = rng.uniform(0.0, spacing, 2)
    t = rng.uniform(-drift, drift, (n, 2)) if drift > 0 else np.zeros((n, 2))
    sines = rng.uniform(0.0, 1.0, (n, 4, 5))
    gen = torch.Generator(device=DEVICE).manual_seed(seed)
    y = torch.arange(height, device=DEVICE, dtype=torch.float32)[None, :, None]
    x = torch.arange(width, device=DEVICE, dtype=torch.float32)[None, None, :]
    shift = torch.tensor(t, device=DEVICE, dtype=torch.float32)
    q = torch.tensor(sines, device=DEVICE, dtype=torch.float32)
    frames = torch.empty((n, height, width), device=DEVICE, dtype=torch.float32)
    chunk = max(1, (1 << 23) // (height * width))
    scale = None
    for k in range(0, n, chunk):
        s, w = shift[k:k + chunk, :, None, None], q[k:k + chunk, :, :, None, None]
        fx, fy = x - s[:, 0], y - s[:, 1]
        for m in range(4 if warp > 0 else 0):
            alpha, wave = w[:, m, 0] * (warp / 4), 32.0 + 96.0 * w[:, m, 1]
            an, ae, ph = (2 * math.pi * w[:, m, j] for j in (2, 3, 4))
            v = alpha * torch.sin(2 * math.pi * (torch.cos(an) * x + torch.sin(an) * y) / wave + ph)
            fx, fy = fx - torch.cos(ae) * v, fy - torch.sin(ae) * v
        fx, fy = (fx - origin[0]) / spacing, (fy - origin[1]) / spacing
        ix, iy = torch.floor(fx), torch.floor(fy)
        rx, ry = (fx - ix) * spacing, (fy - iy) * spacing
        at = (iy.long() + pad) * nx + ix.long() + pad
        clean = 0.0
        for dy in (-1, 0, 1, 2):
            row = 0.0
            for dx in (-1, 0, 1, 2):
                row = row + amps[at + (dy * nx + dx)] * torch.exp((rx - spacing * dx) ** 2 * (-0.5 / sigma ** 2))
            clean = clean + row * torch.exp((ry - spacing * dy) ** 2 * (-0.5 / sigma ** 2))
        if scale is None:
            scale = counts / float(clean[0].mean())
        frames[k:k + chunk] = torch.poisson(clean * scale, generator=gen)
    return frames, shift


def motion(side):
    """Largest drift and warp (px) of the frames of a side."""
    return (2.0, 0.0) if side < 128 else (4.0, 1.0) if side < 512 else (8.0, 1.5)


def smooth_fields(seed, n, height, width, size):
    """[n, 2, height, width] smooth random displacements of about `size` px."""
    gen = torch.Generator(device=DEVICE).manual_seed(seed + 17)
    coarse = torch.randn((n, 2, 6, 6), device=DEVICE, generator=gen) * (0.7 * size)
    return F.interpolate(coarse, size=(height, width), mode="bicubic", align_corners=True)


def net_samples(seed, batch):
    """Network inputs (the reference and the template of a pair, 512-pixel frames restricted to
    128 pixels, mean 0 and sigma 1) and targets (displacements in cells), [batch, 128, 128, 2]."""
    frames, t = blob_frames(seed, batch + 1, 512, 512, 8.0, 1.5, 5.0)
    small = F.avg_pool2d(frames[:, None], 4)[:, 0]
    small = (small - small.mean((1, 2), keepdim=True)) / small.std((1, 2), keepdim=True)
    x = torch.stack([small[:-1], small[1:]], -1).contiguous()
    move = ((t[1:] - t[:-1]) / 4)[:, :, None, None] + smooth_fields(seed, batch, 128, 128, 0.2)
    return x, move.permute(0, 2, 3, 1).contiguous()


def inputs(case, seed):
    """The case's inputs alone (device tensors)."""
    kind = case["kind"]
    if kind in ("pair", "pairs", "series", "rigid", "refine"):
        side = case["side"]
        drift, warp = motion(side)
        n = {"pair": 2, "pairs": case.get("pairs", 0) + 1}.get(kind) or case["frames"]
        frames, t = blob_frames(seed, n, side, side, drift, 0.0 if kind == "rigid" else warp,
                                case["counts"])
        s = {"frames": frames}
        if kind == "pair":
            # a guess near the solution: the pair's drift with a smooth error
            s["guess"] = ((t[1] - t[0])[:, None, None] + smooth_fields(seed, 1, side, side, 0.5)[0]
                          ).contiguous() if case["init"] else None
        if kind == "refine":
            u = (t - t[:1])[:, :, None, None] + smooth_fields(seed, n, side, side, 0.3)
            u[0] = 0
            s["u"] = u.contiguous()
        return s
    if kind == "batch":
        return {"series": [blob_frames(seed * 16 + j, n, side, side, *motion(side), case["counts"])[0]
                           for j, (side, n) in enumerate(shapes_of(case))]}
    if kind == "average":
        n, h, w = case["frames"], case["height"], case["width"]
        frames, t = blob_frames(seed, n, h, w, 8.0, 0.0, 5.0)
        u = torch.empty((n, 2, h, w), device=DEVICE)
        for k in range(0, n, 32):
            u[k:k + 32] = (t[k:k + 32] - t[:1])[:, :, None, None] + smooth_fields(
                seed + k, min(32, n - k), h, w, 1.0)
        u[0] = 0
        return {"frames": frames, "u": u}
    x, target = net_samples(seed, case["batch"])
    return {"x": x, "target": target}


def shapes_of(case):
    return list(zip(map(int, case["sides"].split(",")), map(int, case["lengths"].split(","))))


def trained_net():
    net = P.WarmStartNet()
    net.load(WEIGHTS)
    return net


def prepare(case, seed):
    s = dict(inputs(case, seed), case=case)
    kind = case["kind"]
    if kind in ("forward", "gradients") or case.get("start", "cold") != "cold":
        s["net"] = trained_net()
    if kind in ("pair", "pairs", "series", "rigid", "refine"):
        s["params"] = P.Params(levels=case["levels"], scan=case.get("scan", "brent_kung"),
                               warm_start=int(case.get("start", "cold") != "cold"))
    if kind == "pairs":
        s["ref"], s["tmpl"] = np.arange(case["pairs"]), np.arange(1, case["pairs"] + 1)
    if kind == "batch":
        s["params"] = P.Params(warm_start=0)
        s["levels"] = [levels_of(side) for side, _ in shapes_of(case)]
    if kind == "refine":
        s["work"] = torch.empty_like(s["u"])
    return s


# ---- one pass ---------------------------------------------------------------------------------

def steps_of(stats):
    return np.array([s.iters for s in stats], dtype=np.int64)


def run(s):
    kind = s["case"]["kind"]
    if kind == "pair":
        u, st = P.register_pair(s["frames"][0], s["frames"][1], u_init=s["guess"],
                                params=s["params"])
        return {"u": u, "steps": steps_of([st])}
    if kind == "pairs":
        u, st = P.register_pairs(s["frames"], s["ref"], s["tmpl"], params=s["params"])
        return {"u": u, "steps": steps_of(st)}
    if kind == "series":
        if "net" in s:
            P.set_warm_start(s["net"], mode=s["case"]["start"])
        u, st, _ = P.prefix_register_series(s["frames"], params=s["params"])
        return {"u": u, "node_steps": st.node_steps, "flags": st.flags_or}
    if kind == "batch":
        us, st, _ = P.register_series_batch(s["series"], params=s["params"], levels=s["levels"])
        return {"u": us, "node_steps": [x.node_steps for x in st]}
    if kind == "rigid":
        p, st = P.prefix_register_series_rigid(s["frames"], params=s["params"])
        return {"p": p, "node_steps": st.node_steps}
    if kind == "refine":
        s["work"].copy_(s["u"])  # the procedure refines in place
        u, avg, st = P.series_average_refine(s["frames"], s["work"], passes=1, params=s["params"])
        return {"u": u, "avg": avg, "steps": steps_of(st[0])}
    if kind == "average":
        return {"avg": P.series_average(s["frames"], s["u"])}
    if kind == "forward":
        return {"y": s["net"].forward(s["x"])}
    loss, grad = s["net"].gradients(s["x"], s["target"])
    return {"loss": np.float32(loss), "grad": grad}


# ---- what a pass cannot do without --------------------------------------------------------------

CONV = [(2, 64, 64), (64, 128, 32), (128, 256, 16), (384, 128, 32), (192, 64, 64), (66, 2, 128)]


def work(case):
    """Bytes: inputs read once, results written once. Flops: for a registration one energy and
    one gradient on every node of its frame (it takes as many more as its descent needs); for the
    network its products."""
    kind = case["kind"]
    per_node = 250.0  # four bilinear samples with gradients and the sums over them
    if kind == "pair":
        px = case["side"] ** 2
        return {"bytes": (16.0 + 8.0 * case["init"]) * px, "flops": per_node * px}
    if kind == "pairs":
        px = case["side"] ** 2
        return {"bytes": (4.0 * (case["pairs"] + 1) + 8.0 * case["pairs"]) * px,
                "flops": per_node * case["pairs"] * px}
    if kind in ("series", "batch"):
        px = sum(n * s * s for s, n in (shapes_of(case) if kind == "batch"
                                        else [(case["side"], case["frames"])]))
        return {"bytes": 12.0 * px, "flops": 2 * per_node * px}
    if kind == "rigid":
        px = case["frames"] * case["side"] ** 2
        return {"bytes": 4.0 * px, "flops": 2 * per_node * px}
    if kind == "refine":
        px = case["frames"] * case["side"] ** 2
        return {"bytes": 20.0 * px, "flops": per_node * px}
    if kind == "average":
        px = case["height"] * case["width"]
        return {"bytes": (12.0 * case["frames"] + 4.0) * px, "flops": 16.0 * case["frames"] * px}
    fwd = sum(2.0 * 9 * ci * co * h * h for ci, co, h in CONV) * case["batch"]
    io = 4.0 * 128 * 128 * 2 * case["batch"]
    if kind == "forward":
        return {"bytes": 2 * io, "flops": fwd}
    return {"bytes": 2 * io, "flops": 3 * fwd - 2.0 * 9 * 2 * 64 * 64 * 64 * case["batch"]}


# ---- the same results in FP64 -------------------------------------------------------------------

GAUSS = 0.5 - 0.5 / math.sqrt(3.0)


def restrict64(f):
    """Full weighting to the next coarser level, weights renormalised at the border; [c, n, n]."""
    w = torch.tensor([1.0, 2.0, 1.0], device=f.device, dtype=f.dtype)
    k = (w[:, None] * w[None, :])[None, None]
    num = F.conv2d(F.pad(f[:, None], (1, 1, 1, 1)), k, stride=2)
    den = F.conv2d(F.pad(torch.ones_like(f[:1, None]), (1, 1, 1, 1)), k, stride=2)
    return (num / den)[:, 0]


def at_gauss(f):
    """[..., n, n] nodal values -> [4, ..., n-1, n-1] at the 2x2 Gauss points of each element."""
    out = []
    for e in (GAUSS, 1 - GAUSS):
        r = f[..., :-1, :] * (1 - e) + f[..., 1:, :] * e
        out += [r[..., :-1] * (1 - x) + r[..., 1:] * x for x in (GAUSS, 1 - GAUSS)]
    return torch.stack(out)


def sample64(t, x, y):
    """Bilinear samples of nodal t [n, n] at (x, y) in cells, clamped to the frame."""
    n = t.shape[0]
    x, y = x.clamp(0, n - 1), y.clamp(0, n - 1)
    ix, iy = (v.detach().floor().clamp(max=n - 2) for v in (x, y))
    fx, fy = x - ix, y - iy
    i = (iy * n + ix).long()
    a, b, c, d = (t.reshape(-1)[i + o] for o in (0, 1, n, n + 1))
    return (a * (1 - fx) + b * fx) * (1 - fy) + (c * (1 - fx) + d * fx) * fy


def register64(ref, tmpl, levels, guess, p):
    """Pairwise registration in FP64: [2, side, side] px and the accepted steps per level."""
    side = ref.shape[0]
    L = side.bit_length() - 1
    top = (1 << L) + 1

    def nodes(v):
        v = v.double()
        return v if side == top else F.pad(v[:, None], (0, 1, 0, 1), mode="replicate")[:, 0]

    def pyramid(v):
        out = {L: nodes(v)}
        for l in range(L, L - levels + 1, -1):
            out[l - 1] = restrict64(out[l])
        return out

    f = pyramid(torch.stack([ref, tmpl]))
    g = pyramid(guess / (top - 1)) if guess is not None else None
    counts, u = [], None
    for l in range(L - levels + 1, L + 1):
        n = (1 << l) + 1
        h = 1.0 / (n - 1)
        q = at_gauss(f[l])
        mean = q.mean((0, 2, 3))
        sig = ((q * q).mean((0, 2, 3)) - mean * mean).sqrt()
        R, T = (f[l] - mean[:, None, None]) / sig[:, None, None]
        rq = at_gauss(R)
        if u is None:
            u = g[l] if g is not None else torch.zeros((2, n, n), device=ref.device,
                                                       dtype=torch.float64)
        else:
            u = F.interpolate(u[None], size=(n, n), mode="bilinear", align_corners=True)[0]
        cell = torch.arange(n - 1, device=ref.device, dtype=torch.float64)
        off = torch.tensor([GAUSS, 1 - GAUSS], device=ref.device, dtype=torch.float64)
        gx = (cell[None, None, :] + off.repeat(2)[:, None, None])
        gy = (cell[None, :, None] + off.repeat_interleave(2)[:, None, None])

        def energy(v):
            w = at_gauss(v) * (n - 1)
            t = sample64(T, gx + w[:, 0], gy + w[:, 1])
            m = t.mean()
            ncc = ((rq * t).mean() - m * rq.mean()) / ((t * t).mean() - m * m).sqrt()
            dx, dy = v[:, :, 1:] - v[:, :, :-1], v[:, 1:] - v[:, :-1]
            one = lambda d0, d1: ((d0 * d0 + d0 * d1 + d1 * d1) / 3).sum()
            return -ncc + 0.5 * p.lam * (one(dx[:, :-1], dx[:, 1:]) + one(dy[:, :, :-1], dy[:, :, 1:]))

        c = (p.beta * h) ** 2
        S = torch.diag(torch.full((n,), 2 * h / 3 + 2 * c / h, dtype=torch.float64))
        S[0, 0] = S[-1, -1] = h / 3 + c / h
        S += torch.diag(torch.full((n - 1,), h / 6 - c / h, dtype=torch.float64), 1)
        S += torch.diag(torch.full((n - 1,), h / 6 - c / h, dtype=torch.float64), -1)
        Si = torch.linalg.inv(S).to(ref.device)
        E, tau_prev, done = float(energy(u)), math.inf, 0
        while done < p.iter_max:
            v = u.clone().requires_grad_(True)
            G, = torch.autograd.grad(energy(v), v)
            d = torch.stack([Si @ G[0] @ Si, Si @ G[1] @ Si])
            gtd, dmax = float((G * d).sum()), float(d.abs().max())
            if not gtd > 0 or not dmax > 0:
                break
            tau_max = p.step_cap * h / dmax
            tau = min(tau_prev * 2 ** p.ladder_k, tau_max)
            low, rung, took = p.tau_min_rel * tau_max, 0, None
            while rung % (2 * p.ladder_k + 1) or tau >= low:
                e = float(energy(u - tau * d))
                if e <= E - p.armijo_sigma * tau * gtd:
                    took = e
                    break
                tau, rung = tau / 2, rung + 1
            if took is None:
                break
            u, tau_prev, done, drop, E = u - tau * d, tau, done + 1, E - took, took
            if drop < p.eps:
                break
        counts.append(done)
    return (u * (top - 1))[:, :side, :side].contiguous(), counts


def conv64(x, w, b, stride):
    """3x3 convolution, padding 1, as a matrix product; x [B, C, H, W], w [O, 9 C]."""
    n, _, h, _ = x.shape
    cols = F.unfold(x, 3, padding=1, stride=stride)  # [B, C 9, P], channel-major
    y = torch.matmul(w, cols) + b[:, None]
    return y.reshape(n, w.shape[0], h // stride, h // stride)


def read_weights():
    with open(WEIGHTS, "rb") as f:
        head = int.from_bytes(f.read(8), "little")
        at = json.loads(f.read(head))["params"]["data_offsets"]
        data = f.read()
    return np.frombuffer(data[at[0]:at[1]], dtype=np.float32)


def net_layout():
    """Per layer: offset of the weights, their columns used and stored, offset of the bias."""
    out, at = [], 0
    for j, (ci, co, _) in enumerate(CONV):
        used = 9 * ci
        kept = 64 if j == 0 else used if j == 5 else (used + 31) // 32 * 32
        out.append((at, used, kept, at + co * kept))
        at += co * kept + co
    return out, at


def net64(x, params, want_grad, target=None, margin=4):
    """The network in FP64 with its BF16 weights: outputs, or the loss and its gradient."""
    layers, leaves = [], []
    for (ci, co, _), (w0, used, kept, b0) in zip(CONV, net_layout()[0]):
        w = torch.tensor(params[w0:w0 + co * kept].copy(), device=x.device).bfloat16().double()
        w = w.reshape(co, kept)[:, :used].clone().requires_grad_(want_grad)
        b = torch.tensor(params[b0:b0 + co].copy(), device=x.device).double().requires_grad_(want_grad)
        leaves.append((w, b))
        # stored tap-major (dy, dx, channel); the products below are channel-major
        layers.append((w.reshape(co, 9, ci).transpose(1, 2).reshape(co, 9 * ci), b))
    up = lambda v: v.repeat_interleave(2, 2).repeat_interleave(2, 3)

    def forward(v):
        v = v.bfloat16().double().permute(0, 3, 1, 2)
        a1 = conv64(v, *layers[0], 2).relu()
        a2 = conv64(a1, *layers[1], 2).relu()
        a3 = conv64(a2, *layers[2], 2).relu()
        a4 = conv64(torch.cat([up(a3), a2], 1), *layers[3], 1).relu()
        a5 = conv64(torch.cat([up(a4), a1], 1), *layers[4], 1).relu()
        return conv64(torch.cat([up(a5), v], 1), *layers[5], 1).permute(0, 2, 3, 1)

    if not want_grad:
        with torch.no_grad():
            return torch.cat([forward(x[k:k + 8]) for k in range(0, x.shape[0], 8)])
    loss, count = 0.0, 0
    inner = slice(margin, 128 - margin)
    total = x.shape[0] * 2 * (128 - 2 * margin) ** 2
    for k in range(0, x.shape[0], 8):
        part = ((forward(x[k:k + 8]) - target[k:k + 8].double())[:, inner, inner] ** 2).sum() / total
        part.backward(retain_graph=True)
        loss += part.item()
    grad = np.zeros(net_layout()[1])
    for (w, b), (ci, co, _), (w0, used, kept, b0) in zip(leaves, CONV, net_layout()[0]):
        m = np.zeros((co, kept))
        m[:, :used] = w.grad.cpu().numpy()
        grad[w0:w0 + co * kept] = m.ravel()
        grad[b0:b0 + co] = b.grad.cpu().numpy()
    return loss, grad


def exact(case, seed):
    kind = case["kind"]
    if kind in ("series", "batch", "rigid", "refine"):
        # chains of registrations: minutes in FP64 (and every stop decision is a branch)
        return None
    if kind in ("pair", "pairs"):
        count, px = case.get("pairs", 1), case["side"] ** 2
        if count * px > 16 * 257 ** 2:
            return None  # over 20 s
        s, p = inputs(case, seed), P.Params(levels=case["levels"])
        got = [register64(s["frames"][k], s["frames"][k + 1], case["levels"], s.get("guess"), p)[0]
               for k in range(count)]
        return {"u": torch.stack(got) if kind == "pairs" else got[0], "steps": None}
    s = inputs(case, seed)
    if kind == "average":
        n, h, w = s["frames"].shape
        y, x = torch.meshgrid(*(torch.arange(v, device=DEVICE, dtype=torch.float64) for v in (h, w)),
                              indexing="ij")
        out = torch.zeros((h, w), device=DEVICE, dtype=torch.float64)
        for f, u in zip(s["frames"], s["u"].unbind()):
            px, py = (x + u[0].double()).clamp(0, w - 1), (y + u[1].double()).clamp(0, h - 1)
            ix, iy = px.floor().clamp(max=w - 2), py.floor().clamp(max=h - 2)
            fx, fy = px - ix, py - iy
            i, g = (iy * w + ix).long(), f.double().reshape(-1)
            out += (g[i] * (1 - fx) + g[i + 1] * fx) * (1 - fy) + (
                g[i + w] * (1 - fx) + g[i + w + 1] * fx) * fy
        return {"avg": out / n}
    if kind == "forward":
        return {"y": net64(s["x"], read_weights(), False)}
    loss, grad = net64(s["x"], read_weights(), True, s["target"])
    return {"loss": np.float64(loss), "grad": grad}

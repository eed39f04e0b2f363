"""The work that users of this package have it do, as cases that can be timed and checked.

    listed()            named cases over the range of real use
    draw(rng)           one more case of the same ranges
    prepare(case, seed) inputs, plans and networks a program holds before the call
    run(state)          one pass through the public entry points; its outputs
    work(case)          bytes and operations one pass cannot do without
    exact(case, seed)   the outputs in 64 bits, from plain torch

Kinds of case:

    pair      forward projection of an image, then the adjoint of the result (one operator
              application of an iterative reconstruction)
    fbp       filtered adjoint of a measured sinogram
    slices    forward and adjoint of several slices that share one geometry
    uneven    forward and adjoint of slices of different sizes as one Batch
    solve     a basis-pursuit reconstruction with a fixed iteration budget
    project   projection of an image-sized vector onto the l1 ball
    ring      ring filter of a sinogram
    net       the warm-start network's forward pass
    train     training steps of the warm-start network, then its weights
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1009_1380_amd import Batch, Plan, WarmStartNet, project_l1

DEV = "cuda"
# image sides and detector counts used in earnest (all are supported FFT lengths)
SIDES = (64, 80, 96, 128, 160, 192, 256, 320, 384, 512, 640, 768, 1024, 1280, 1536, 2048, 2560)
CHANNELS = ((1, 32), (32, 64), (64, 128), (128, 256), (256, 128), (128, 64), (64, 32), (32, 1))
SNR = 10.0 ** (-30.0 / 20.0)          # measured sinograms carry noise at 30 dB


def listed():
    return [
        # a small slice, as in interactive work and parity runs: launch latency counts
        {"name": "pair_128", "kind": "pair", "n": 128, "views": 180, "det": 128, "W": 6},
        # few-view slice of the warm-start workload
        {"name": "pair_512_90v", "kind": "pair", "n": 512, "views": 90, "det": 512, "W": 6},
        # detector unlike the image side, an odd view count and the widest kernel
        {"name": "pair_ragged", "kind": "pair", "n": 1536, "views": 361, "det": 1280, "W": 8},
        # full-size slice, the benchmark's workload
        {"name": "pair_2560", "kind": "pair", "n": 2560, "views": 1024, "det": 2560, "W": 6},
        # quick-look reconstruction of the reduced-view scan
        {"name": "fbp_1024", "kind": "fbp", "n": 1024, "views": 128, "det": 1024, "W": 6},
        # a stack of a volume's slices under one plan
        {"name": "slices_512x8", "kind": "slices", "n": 512, "views": 180, "det": 512, "W": 6, "count": 8},
        # a mixed queue of slices, as a batch
        {"name": "uneven_16", "kind": "uneven", "count": 16, "lo": 512, "hi": 2560, "mix": 1},
        # reduced-view reconstruction under an iteration budget
        {"name": "solve_1024", "kind": "solve", "n": 1024, "views": 128, "det": 1024, "iters": 16, "warm": False},
        # the solver's projection on its own, as in a user's own proximal loop
        {"name": "project_1024", "kind": "project", "numel": 1024 * 1024, "tau": 0.1},
        # ring removal on a full-size sinogram
        {"name": "ring_1024x2560", "kind": "ring", "views": 1024, "det": 2560},
        # start image of one slice
        {"name": "net_512", "kind": "net", "batch": 1, "height": 512, "width": 512},
        # fine-tuning on mini-batches of eight slices, then a checkpoint of the weights
        {"name": "train_512x8", "kind": "train", "batch": 8, "height": 512, "width": 512, "steps": 4},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("pair", "pair", "fbp", "slices", "uneven", "solve", "project", "ring", "net", "train"))
    n = min(SIDES, key=lambda s: abs(math.log(s / _log(rng, 64, 2560))))
    det = rng.choice([s for s in SIDES if n / 2 <= s <= 2 * n])
    if kind in ("pair", "fbp"):
        return {"kind": kind, "n": n, "views": _log(rng, 16, 1024), "det": det, "W": rng.choice((4, 6, 6, 8))}
    if kind == "slices":
        n = min(n, 1024)
        return {"kind": kind, "n": n, "views": _log(rng, 16, 361), "det": n, "W": 6, "count": rng.randint(2, 12)}
    if kind == "uneven":
        lo = rng.choice((128, 256, 512))
        return {"kind": kind, "count": rng.randint(3, 16), "lo": lo, "hi": rng.choice((1024, 1536, 2560)),
                "mix": rng.randint(2, 1 << 20)}
    if kind == "solve":
        n = min(n, 1024)
        return {"kind": kind, "n": n, "views": _log(rng, 24, 128), "det": n, "iters": rng.randint(4, 14),
                "warm": rng.random() < 0.5}
    if kind == "project":
        return {"kind": kind, "numel": 4 * _log(rng, 1 << 8, 1 << 20), "tau": round(rng.uniform(0.01, 0.9), 3)}
    if kind == "ring":
        return {"kind": kind, "views": _log(rng, 16, 1024), "det": rng.choice(SIDES)}
    h, w = 8 * _log(rng, 6, 64), 8 * _log(rng, 6, 64)
    if kind == "net":
        return {"kind": kind, "batch": rng.randint(1, 8), "height": h, "width": w}
    return {"kind": kind, "batch": rng.randint(1, 8), "height": h, "width": w, "steps": rng.randint(1, 4)}


# ------------------------------------------------------------------ inputs


def _rng(seed, salt):
    return np.random.default_rng([int(seed), int(salt)])


def _noise(seed, salt, shape):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 1009 + int(salt))
    return torch.randn(shape, generator=g, device=DEV, dtype=torch.float32)


def _angles(views):
    return np.arange(views, dtype=np.float64) * (np.pi / views)


def _disks(seed, salt, n, count=24):
    """Disks inside the inscribed circle: centre, radius, density."""
    r = _rng(seed, salt)
    rad = r.uniform(0.02, 0.12, count) * n
    dist = np.sqrt(r.uniform(0.0, 1.0, count)) * (n / 2 - 2 - rad)
    phi = r.uniform(0.0, 2 * np.pi, count)
    return list(zip(dist * np.cos(phi), dist * np.sin(phi), rad, r.uniform(0.5, 1.0, count)))


def _image(seed, salt, n, m=None):
    """Slice through spheres (n x m, m = n by default) with pixel noise."""
    m = n if m is None else m
    y = (torch.arange(n, device=DEV, dtype=torch.float32) - n // 2)[:, None]
    x = (torch.arange(m, device=DEV, dtype=torch.float32) - m // 2)[None, :]
    img = 1e-2 * _noise(seed, salt, (n, m))
    for cx, cy, r, rho in _disks(seed, salt, min(n, m)):
        d = torch.sqrt((x - cx) ** 2 + (y - cy) ** 2)
        img += rho * torch.clamp(r - d + 0.5, 0.0, 1.0)
    return img


def _sinogram(seed, salt, n, views, det):
    """Line integrals of the disks, with detector gains (ring stripes) and noise."""
    ang = torch.from_numpy(_angles(views)).to(DEV)[:, None]
    s = (torch.arange(det, device=DEV, dtype=torch.float64) - det // 2)[None, :]
    out = torch.zeros((views, det), device=DEV, dtype=torch.float64)
    for cx, cy, r, rho in _disks(seed, salt, min(n, det)):
        t = s - (cx * torch.cos(ang) + cy * torch.sin(ang))
        out += rho * 2.0 * torch.sqrt(torch.clamp(r * r - t * t, min=0.0))
    scale = out.square().mean().sqrt()
    gains = torch.from_numpy(_rng(seed, salt + 1).normal(1.0, 0.02, det)).to(DEV)
    return (out * gains[None, :] + SNR * scale * _noise(seed, salt, (views, det))).float()


def _shapes(case):
    """Sides and view counts of an uneven batch."""
    r = _rng(case["mix"], 7)
    sides = [s for s in SIDES if case["lo"] <= s <= case["hi"]]
    return [(int(r.choice(sides)), int(np.exp(r.uniform(np.log(45), np.log(720))))) for _ in range(case["count"])]


def _weights(seed):
    """Parameters like a trained network's: He-scaled layers, a small last one."""
    r = _rng(seed, 11)
    parts = []
    for k, (cin, cout) in enumerate(CHANNELS):
        sd = math.sqrt(2.0 / (9 * cin)) * (0.1 if k == len(CHANNELS) - 1 else 1.0)
        parts += [sd * r.standard_normal(9 * cin * cout), 0.01 * r.standard_normal(cout)]
    return np.concatenate(parts).astype(np.float32)


def _batches(case, seed):
    """Network inputs: noisy slices; targets: the slices without the noise."""
    b, h, w = case["batch"], case["height"], case["width"]
    out = []
    for k in range(case.get("steps", 1)):
        t = torch.stack([_image(seed, 100 * k + i, h, w) for i in range(b)])
        out.append((t + 0.1 * _noise(seed, 5000 + k, (b, h, w)), t))
    return out


LR = 1e-5          # fine-tuning rate


# ------------------------------------------------------------------ one pass


def prepare(case, seed):
    c, kind = case, case["kind"]
    if kind == "pair":
        return {"case": c, "plan": Plan(c["n"], _angles(c["views"]), c["det"], 2.0, c["W"]), "x": _image(seed, 1, c["n"])}
    if kind == "fbp":
        return {"case": c, "plan": Plan(c["n"], _angles(c["views"]), c["det"], 2.0, c["W"]),
                "y": _sinogram(seed, 1, c["n"], c["views"], c["det"])}
    if kind == "slices":
        return {"case": c, "plan": Plan(c["n"], _angles(c["views"]), c["det"], 2.0, c["W"]),
                "x": torch.stack([_image(seed, 2 + i, c["n"]) for i in range(c["count"])])}
    if kind == "uneven":
        shapes = _shapes(c)
        plans = [Plan(n, _angles(v), n) for n, v in shapes]
        return {"case": c, "plans": plans, "batch": Batch(plans), "x": [_image(seed, 2 + i, n) for i, (n, _) in enumerate(shapes)],
                "sino": [torch.empty((v, n), device=DEV) for n, v in shapes],
                "back": [torch.empty((n, n), device=DEV) for n, _ in shapes]}
    if kind == "solve":
        plan = Plan(c["n"], _angles(c["views"]), c["det"])
        y = _sinogram(seed, 1, c["n"], c["views"], c["det"])
        s = {"case": c, "plan": plan, "y": y, "sigma": SNR * float(torch.linalg.norm(plan.ring_filter(y).double()))}
        s["x0"] = 0.9 * plan.fbp(y) if c["warm"] else None
        return s
    if kind == "project":
        # an image-sized gradient step: many small values, few large ones
        v = _noise(seed, 1, (c["numel"],)) ** 3
        return {"case": c, "v": v, "tau": c["tau"] * float(v.abs().double().sum())}
    if kind == "ring":
        plan = Plan(64, _angles(c["views"]), c["det"])
        return {"case": c, "plan": plan, "y": _sinogram(seed, 1, c["det"], c["views"], c["det"])}
    net = WarmStartNet(c["batch"], c["height"], c["width"], seed=0)
    net.set_params(_weights(seed))
    return {"case": c, "net": net, "data": _batches(c, seed)}


def run(s):
    kind = s["case"]["kind"]
    if kind == "pair":
        y = s["plan"].forward(s["x"])
        return {"sino": y, "back": s["plan"].adjoint(y)}
    if kind == "fbp":
        return s["plan"].fbp(s["y"])
    if kind == "slices":
        y = s["plan"].forward_batched(s["x"])
        return {"sino": y, "back": s["plan"].adjoint_batched(y)}
    if kind == "uneven":
        s["batch"].forward(s["x"], s["sino"])
        s["batch"].adjoint(s["sino"], s["back"])
        return {"sino": s["sino"], "back": s["back"]}
    if kind == "solve":
        x, st = s["plan"].solve_bpdn(s["y"], s["sigma"], x0=s["x0"], opt_tol=1e-3, max_iter=s["case"]["iters"])
        return {"x": x, "rnorm": st["rnorm"], "tau": st["tau"]}
    if kind == "project":
        out, lam = project_l1(s["v"], s["tau"])
        return {"out": out, "lam": lam}
    if kind == "ring":
        return s["plan"].ring_filter(s["y"])
    if kind == "net":
        return s["net"].forward(s["data"][0][0])
    for x, t in s["data"]:
        pred = torch.empty_like(x)
        loss = s["net"].train_step(x, t, LR, pred=pred)
    return {"pred": pred, "loss": loss, "params": s["net"].get_params()}


# ------------------------------------------------------------------ what a pass cannot do without


def _one(n, views, det, W):
    """Operations of one direction: two-dimensional FFT onto the doubled grid (real data, the
    zero half skipped in one axis), footprint sums of half the samples, ray FFTs."""
    g = 2 * n
    fft2 = 2.5 * g * math.log2(g) * n + 5.0 * g * math.log2(g) * (n + 1)
    return fft2 + 0.5 * views * det * W * W * 4.0 + 2.5 * views * det * math.log2(det)


def _conv_flops(case):
    b, h, w = case["batch"], case["height"], case["width"]
    scale = (1, 4, 16, 64, 16, 4, 1, 1)
    return [2.0 * 9 * ci * co * b * h * w / s for (ci, co), s in zip(CHANNELS, scale)]


def work(case):
    c, kind = case, case["kind"]
    if kind in ("pair", "slices"):
        k, io = c.get("count", 1), 4 * (c["n"] ** 2 + c["views"] * c["det"])
        return {"bytes": 2 * k * io, "flops": 2 * k * _one(c["n"], c["views"], c["det"], c["W"])}
    if kind == "fbp":
        return {"bytes": 4 * (c["n"] ** 2 + c["views"] * c["det"]), "flops": _one(c["n"], c["views"], c["det"], c["W"])}
    if kind == "uneven":
        sh = _shapes(c)
        return {"bytes": sum(8 * (n * n + v * n) for n, v in sh), "flops": sum(2 * _one(n, v, n, 6) for n, v in sh)}
    if kind == "solve":
        # per iteration: one forward and one adjoint, the iterate and gradient read and written
        per = 2 * _one(c["n"], c["views"], c["det"], 6)
        return {"bytes": c["iters"] * 4 * (4 * c["n"] ** 2 + 4 * c["views"] * c["det"]), "flops": c["iters"] * per}
    if kind == "project":
        return {"bytes": 8 * c["numel"], "flops": 4 * c["numel"]}
    if kind == "ring":
        return {"bytes": 8 * c["views"] * c["det"], "flops": 2 * c["views"] * c["det"]}
    px, weights = c["batch"] * c["height"] * c["width"], sum(9 * ci * co + co for ci, co in CHANNELS)
    fl = _conv_flops(c)
    if kind == "net":
        return {"bytes": 8 * px + 4 * weights, "flops": sum(fl)}
    # forward, weight gradients, data gradients of all layers but the first
    return {"bytes": c["steps"] * (12 * px + 24 * weights), "flops": c["steps"] * (2 * sum(fl) + sum(fl[1:]))}


# ------------------------------------------------------------------ the outputs in 64 bits


class _Grid:
    """Gridding forward and adjoint in float64: deapodize, zero-pad, FFT, Kaiser-Bessel
    footprint sums, ray FFTs; the adjoint is the transpose."""

    def __init__(self, n, ang, det, W):
        self.n, self.det, self.W, self.G = n, det, W, 2 * n
        beta = math.pi * math.sqrt((W / 2.0) ** 2 * 1.5 ** 2 - 0.8)
        f = (np.arange(n, dtype=np.float64) - n // 2) / self.G
        z2 = (beta * beta - (math.pi * W * f) ** 2).astype(np.complex128)
        z = np.sqrt(z2)
        psi = (np.sinh(z) / z).real * W / np.i0(beta)
        self.inv = torch.from_numpy(1.0 / psi).to(DEV)
        self.beta, self.i0b = beta, torch.special.i0(torch.tensor(beta, dtype=torch.float64, device=DEV))
        q = np.arange(det, dtype=np.int64) - det // 2
        fq = (self.G * q) / float(det)
        c = np.array([math.cos(a) for a in ang])
        s = np.array([math.sin(a) for a in ang])
        self.u = torch.from_numpy(fq[None, :] * c[:, None]).to(DEV)
        self.v = torch.from_numpy(fq[None, :] * s[:, None]).to(DEV)
        self.pad = (torch.arange(n, device=DEV) - n // 2) % self.G

    def _phi(self, t):
        r = 2.0 * t / self.W
        w = torch.special.i0(self.beta * torch.sqrt(torch.clamp(1.0 - r * r, min=0.0))) / self.i0b
        return torch.where(t.abs() < self.W / 2.0, w, torch.zeros_like(w))

    def _taps(self):
        bu, bv = torch.floor(self.u), torch.floor(self.v)
        for g in range(-self.W // 2 + 1, self.W // 2 + 1):
            wy = self._phi(self.v - (bv + g))
            rows = (bv.long() + g) % self.G
            for a in range(-self.W // 2 + 1, self.W // 2 + 1):
                yield wy * self._phi(self.u - (bu + a)), rows * self.G + (bu.long() + a) % self.G

    def forward(self, x):
        P = torch.zeros((self.G, self.G), dtype=torch.complex128, device=DEV)
        P[self.pad[:, None], self.pad[None, :]] = (x.double() * self.inv[:, None] * self.inv[None, :]).to(torch.complex128)
        flat = torch.fft.fft2(P).reshape(-1)
        X = torch.zeros(self.u.shape, dtype=torch.complex128, device=DEV)
        for w, idx in self._taps():
            X += w * flat[idx]
        return torch.fft.fftshift(torch.fft.ifft(torch.fft.ifftshift(X, dim=1), dim=1), dim=1).real.contiguous()

    def adjoint(self, y, weights=None):
        Y = torch.fft.fftshift(torch.fft.fft(torch.fft.ifftshift(y.double(), dim=1), dim=1), dim=1) / self.det
        if weights is not None:
            Y = Y * weights[None, :]
        re = torch.zeros(self.G * self.G, dtype=torch.float64, device=DEV)
        im = torch.zeros_like(re)
        for w, idx in self._taps():
            re.index_add_(0, idx.reshape(-1), (w * Y.real).reshape(-1))
            im.index_add_(0, idx.reshape(-1), (w * Y.imag).reshape(-1))
        h = torch.fft.ifft2(torch.complex(re, im).reshape(self.G, self.G)) * (self.G * self.G)
        return h[self.pad[:, None], self.pad[None, :]].real * self.inv[:, None] * self.inv[None, :]


def _ramp(views, det):
    k = np.arange(det) - det // 2
    h = np.where(k % 2 != 0, -1.0 / (np.pi * np.where(k == 0, 1, k)) ** 2, 0.0)
    h[det // 2] = 0.25
    return torch.from_numpy(np.pi / views * np.fft.fftshift(np.fft.fft(np.fft.ifftshift(h)).real)).to(DEV)


def _conv64(x, w, b):
    """3x3 convolution with zero padding as nine matrix products, float64."""
    n, c, h, wd = x.shape
    p = torch.nn.functional.pad(x, (1, 1, 1, 1))
    out = b[None, :, None].expand(n, -1, h * wd)
    for i in range(3):
        for j in range(3):
            t = p[:, :, i:i + h, j:j + wd].reshape(n, c, h * wd)
            out = out + torch.matmul(w[:, :, i, j].contiguous(), t)
    return out.reshape(n, -1, h, wd)


def _net64(params, x):
    layers, off = [], 0
    for ci, co in CHANNELS:
        layers.append((params[off:off + 9 * ci * co].reshape(co, ci, 3, 3), params[off + 9 * ci * co:off + 9 * ci * co + co]))
        off += 9 * ci * co + co
    conv = lambda k, t: _conv64(t, *layers[k])                                              # noqa: E731
    pool = lambda t: 0.25 * (t[..., ::2, ::2] + t[..., 1::2, ::2] + t[..., ::2, 1::2] + t[..., 1::2, 1::2])  # noqa: E731
    up = lambda t: t.repeat_interleave(2, -1).repeat_interleave(2, -2)                      # noqa: E731
    e0 = torch.relu(conv(0, x[:, None]))
    e1 = torch.relu(conv(1, pool(e0)))
    e2 = torch.relu(conv(2, pool(e1)))
    e3 = torch.relu(conv(3, pool(e2)))
    d2 = torch.relu(conv(4, up(e3))) + e2
    d1 = torch.relu(conv(5, up(d2))) + e1
    d0 = torch.relu(conv(6, up(d1))) + e0
    return conv(7, d0)[:, 0] + x


def _project64(v, tau):
    a = v.abs().double().sort(descending=True).values
    cs = a.cumsum(0)
    k = torch.arange(1, a.numel() + 1, device=DEV, dtype=torch.float64)
    rho = int((a * k > cs - tau).sum())
    lam = (cs[rho - 1] - tau) / rho if float(cs[-1]) > tau else torch.zeros((), dtype=torch.float64, device=DEV)
    return {"out": torch.sign(v.double()) * torch.clamp(v.abs().double() - lam, min=0.0), "lam": lam}


def exact(case, seed):
    c, kind = case, case["kind"]
    if kind in ("pair", "fbp", "slices"):
        g = _Grid(c["n"], _angles(c["views"]), c["det"], c["W"])
        if kind == "pair":
            y = g.forward(_image(seed, 1, c["n"]))
            return {"sino": y, "back": g.adjoint(y)}
        if kind == "fbp":
            return g.adjoint(_sinogram(seed, 1, c["n"], c["views"], c["det"]), _ramp(c["views"], c["det"]))
        ys = [g.forward(_image(seed, 2 + i, c["n"])) for i in range(c["count"])]
        return {"sino": torch.stack(ys), "back": torch.stack([g.adjoint(y) for y in ys])}
    if kind == "uneven":
        ys, bs = [], []
        for i, (n, v) in enumerate(_shapes(c)):
            g = _Grid(n, _angles(v), n, 6)
            ys.append(g.forward(_image(seed, 2 + i, n)))
            bs.append(g.adjoint(ys[-1]))
        return {"sino": ys, "back": bs}
    if kind == "solve":
        # the iterates of a nonsmooth method amplify rounding by their discrete choices (line
        # search, active set): no 64-bit value belongs to a given iteration
        return None
    if kind == "project":
        v = _noise(seed, 1, (c["numel"],)) ** 3
        return _project64(v, c["tau"] * float(v.abs().double().sum()))
    if kind == "ring":
        y = _sinogram(seed, 1, c["det"], c["views"], c["det"]).double()
        m = y.mean(dim=0)
        t = (torch.arange(c["det"], device=DEV, dtype=torch.float64) - c["det"] // 2) / (c["det"] // 2)
        q = torch.from_numpy(np.linalg.qr(torch.stack([t ** k for k in range(4)], dim=1).cpu().numpy())[0]).to(DEV)
        return y - (m - q @ (q.T @ m))[None, :]
    p = torch.from_numpy(_weights(seed)).to(DEV).double()
    data = [(x.double(), t.double()) for x, t in _batches(c, seed)]
    if kind == "net":
        with torch.no_grad():
            return _net64(p, data[0][0])
    m, v = torch.zeros_like(p), torch.zeros_like(p)
    for k, (x, t) in enumerate(data, 1):
        p = p.detach().requires_grad_(True)
        grad, loss, pred = torch.zeros_like(p), 0.0, []
        for i in range(x.shape[0]):            # slice by slice: float64 activations are large
            y = _net64(p, x[i:i + 1])
            part = (y - t[i:i + 1]).square().sum() / x.numel()
            grad += torch.autograd.grad(part, p)[0]
            loss, pred = loss + float(part.detach()), pred + [y.detach()]
        m, v = 0.9 * m + 0.1 * grad, 0.999 * v + 0.001 * grad * grad
        p = p.detach() - LR * (m / (1 - 0.9 ** k)) / (torch.sqrt(v / (1 - 0.999 ** k)) + 1e-8)
    return {"pred": torch.cat(pred), "loss": torch.tensor(loss, dtype=torch.float64), "params": p}

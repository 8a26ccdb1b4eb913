"""The work that users have this library do, as cases that can be timed and checked.

Six operations through the package's public entry points:
  fwdinv   ShearletSystem.forward, then inverse (Algorithms 1 and 2);
  layer    ShearletLayer forward and backward (the adjoint) through autograd;
  denoise  ShearletSystem.denoise with per-filter thresholds and kept counts;
  inpaint  UnevenInpainter.run on images of mixed sizes (Algorithm 3);
  apply    ShrinkNet.apply, the learned-shrinkage network on coefficients in hand;
  train    ShrinkNet.train_step, one optimiser step of that network.
"bank" runs forward and inverse of a user's own filter bank (real or complex spectra).

A system is built once per size and kept, as a program keeps it; "tuned" says whether the program
asked for autotune() at its batch (throughput programs do) or took the system as built (one-off calls).
Inputs are cartoons of random ellipses with values in [0, 255] plus noise, made on the GPU from the
seed. Hard thresholds follow the rules of the method and are moved within 2 % into a gap of the
coefficients' magnitudes, so that keep-or-zero decisions do not hang on the last bit of a sum.
"""
import math
import random

import numpy as np
import torch

from paper_2006_04591_amd import ShearletLayer, ShearletSystem, ShrinkNet, UnevenInpainter

DEV = "cuda"


def listed():
    return [
        # the smallest call: one 128 x 128 image, 17 filters, a system straight from build()
        {"name": "fwdinv 128 k17 b1", "op": "fwdinv", "rows": 128, "cols": 128, "scales": 2, "batch": 1, "tuned": False},
        # one 512 x 512 image, 49 filters, untuned: interactive use
        {"name": "fwdinv 512 k49 b1", "op": "fwdinv", "rows": 512, "cols": 512, "scales": 4, "batch": 1, "tuned": False},
        # the throughput workload: 16 images of 512 x 512, 49 filters
        {"name": "fwdinv 512 k49 b16", "op": "fwdinv", "rows": 512, "cols": 512, "scales": 4, "batch": 16, "tuned": True},
        # the largest images that are transformed in batches, untuned
        {"name": "fwdinv 1024 k49 b3", "op": "fwdinv", "rows": 1024, "cols": 1024, "scales": 4, "batch": 3, "tuned": False},
        # a user's own bank of complex spectra (asymmetric kernels) on wide images, an odd batch
        {"name": "bank 256x512 k12 b5", "op": "bank", "rows": 256, "cols": 512, "filters": 12, "batch": 5, "real": False},
        # the fixed layer of a network at its training batch, forward and backward
        {"name": "layer 256 k33 b32", "op": "layer", "rows": 256, "cols": 256, "scales": 3, "batch": 32, "tuned": True},
        # the same on rectangular crops with a ragged batch, untuned
        {"name": "layer 128x256 k17 b7", "op": "layer", "rows": 128, "cols": 256, "scales": 2, "batch": 7, "tuned": False},
        # batched denoising, and three images as they come
        {"name": "denoise 512 k49 b16", "op": "denoise", "rows": 512, "cols": 512, "scales": 4, "batch": 16, "tuned": True},
        {"name": "denoise 256 k33 b3", "op": "denoise", "rows": 256, "cols": 256, "scales": 3, "batch": 3, "tuned": False},
        # inpainting of mixed sizes in one call (the inpainter tunes itself)
        {"name": "inpaint mixed i8", "op": "inpaint", "sizes": "512,256,1024,256,512", "iterations": 8},
        # the learned-shrinkage network: inference, and one training step, on a batch of coefficients
        {"name": "apply 512 k49 b16", "op": "apply", "rows": 512, "cols": 512, "scales": 4, "batch": 16, "tau": False},
        {"name": "train 512 k49 b16", "op": "train", "rows": 512, "cols": 512, "scales": 4, "batch": 16},
    ]


_MOST = 16 * 49 * 512 * 512  # coefficients of the largest listed cases


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 0.5)))))))


def draw(rng):
    op = rng.choice(["fwdinv", "fwdinv", "layer", "denoise", "bank", "inpaint", "apply", "train"])
    if op == "inpaint":
        sizes = [rng.choice([128, 256, 512, 1024]) for _ in range(rng.randint(1, 5))]
        while sum(n * n for n in sizes) > 1024 * 1024 + 2 * 512 * 512:
            sizes.remove(max(sizes))
        return {"op": op, "sizes": ",".join(str(n) for n in sizes), "iterations": rng.randint(2, 8)}
    if op == "bank":
        rows, cols = rng.choice([16, 32, 64, 128, 256, 512, 1024, 2048]), rng.choice([16, 32, 64, 128, 256, 512, 1024, 2048])
        filters = rng.randint(2, 24)
        while rows * cols * filters > 1 << 24:
            filters = (filters + 1) // 2
        return {"op": op, "rows": rows, "cols": cols, "filters": filters,
                "batch": _log_int(rng, 1, max(1, min(64, _MOST // 4 // (filters * rows * cols)))), "real": rng.random() < 0.5}
    rows, cols = rng.choice([(128, 128), (128, 256), (256, 128), (256, 256), (256, 512), (512, 256), (512, 512), (512, 1024), (1024, 512), (1024, 1024)])
    if op in ("apply", "train"):
        rows, cols = min(rows, 512), min(cols, 512)
    scales = rng.choice([2, 3] if min(rows, cols) < 256 else [2, 3, 4])
    c = {"op": op, "rows": rows, "cols": cols, "scales": scales,
         "batch": _log_int(rng, 1, max(1, min(48, _MOST // (_filters(scales) * rows * cols))))}
    if op == "apply":
        c["tau"] = rng.random() < 0.3
    elif op != "train":
        c["tuned"] = rng.random() < 0.5
    return c


# ---------------------------------------------------------------- inputs

def _levels(scales):
    return [(j + 1) // 2 for j in range(1, scales + 1)]


def _filters(scales):
    return 1 + sum(2 ** (s + 2) for s in _levels(scales))


def _images(rows, cols, batch, seed, sigma=0.0):
    """Cartoons of 5 to 10 ellipses, float32 (batch, rows, cols), plus noise of deviation sigma (a number or one per image)."""
    rng = random.Random(seed)
    i = torch.arange(rows, device=DEV, dtype=torch.float32)[:, None]
    j = torch.arange(cols, device=DEV, dtype=torch.float32)[None, :]
    x = torch.zeros((batch, rows, cols), device=DEV)
    m = min(rows, cols)
    for b in range(batch):
        for _ in range(rng.randint(5, 10)):
            di, dj = i - rng.uniform(0, rows), j - rng.uniform(0, cols)
            r0, r1, th, v = rng.uniform(0.05, 0.35) * m, rng.uniform(0.05, 0.35) * m, rng.uniform(0, math.pi), rng.uniform(0, 255)
            c, s = math.cos(th), math.sin(th)
            x[b].masked_fill_(((di * c + dj * s) / r0) ** 2 + ((dj * c - di * s) / r1) ** 2 <= 1, v)
    g = torch.Generator(device=DEV).manual_seed(seed)
    noise = torch.randn(x.shape, generator=g, device=DEV)
    return x + (sigma[:, None, None] if torch.is_tensor(sigma) else sigma) * noise


# ---------------------------------------------------------------- the filters and transforms, in 64 bits

_spectra = {}


def _bank(rows, cols, scales):
    """The filters' real spectra (K, rows, cols) in natural DFT order: the closed forms of the construction."""
    key = (rows, cols, scales)
    if key in _spectra:
        return _spectra[key]
    a = np.linalg.solve([[1, 2, 2, 2, 2], [0, 1, 4, 9, 16], [0, 1, 16, 81, 256], [1, -2, 2, -2, 2], [1, 0, -2, 0, 2]],
                        [1, 0, 0, 0, 0.5 ** 0.5])

    def low(w):  # the 9-tap scaling filter
        return a[0] + 2 * sum(a[n] * torch.cos(n * w) for n in range(1, 5))

    def lows(w, level):
        out = torch.ones_like(w)
        for i in range(level):
            out = out * low(2 ** i * w)
        return out

    def fan(w1, w2):  # the maximally flat fan
        y = 0.5 - (torch.cos(w2) - torch.cos(w1)) / 4
        return (1 - y) ** 4 * sum(math.comb(3 + i, i) * y ** i for i in range(4))

    def shearlet(n1, n2, j, s, k):  # the wavelet along axis 0, the wedge of shear k
        w1 = 2 * math.pi * torch.arange(n1, device=DEV, dtype=torch.float64)[:, None] / n1
        w2 = 2 * math.pi * torch.arange(n2, device=DEV, dtype=torch.float64)[None, :] / n2
        level, u = scales - j + 1, 2 ** s
        band = low(2 ** (level - 1) * w1 + math.pi) * lows(w1, level - 1)
        wedge = 0
        for m in range(u):
            al = (w1 + 2 * math.pi * m) / u
            wedge = wedge + lows(al, s) ** 2 * lows(w2 - k * al, s)
        return band * fan(w1, u * w2 - k * w1) * wedge

    out = []
    for j, s in enumerate(_levels(scales), 1):
        out += [shearlet(rows, cols, j, s, k) for k in range(-2 ** s, 2 ** s + 1)]
        out += [shearlet(cols, rows, j, s, k).T for k in range(1 - 2 ** s, 2 ** s)]
    wr, wc = (2 * math.pi * torch.arange(n, device=DEV, dtype=torch.float64) / n for n in (rows, cols))
    out.append(lows(wr, scales)[:, None] * lows(wc, scales)[None, :])
    _spectra[key] = torch.stack(out)
    return _spectra[key]


def _rms(S):
    return S.abs().square().mean(dim=(1, 2)).sqrt()


def _sh(x, S):
    """Coefficients (B, K, rows, cols) of the images x, float64."""
    return torch.stack([torch.fft.ifft2(torch.fft.fft2(v.double()) * S.conj()).real for v in x])


def _adj(c, S, dual):
    W = S.abs().square().sum(0) if dual else 1.0
    return torch.stack([torch.fft.ifft2((torch.fft.fft2(v.double()) * S).sum(0) / W).real for v in c])


def _in_gap(c, want):
    """Thresholds (K,) within 2 % of `want`, each in the middle of the widest gap there between the magnitudes of its plane of c (K, rows, cols)."""
    K, nb = c.shape[0], 4096
    lo = 0.98 * want
    at = ((c.abs() - lo[:, None, None]) / (0.04 * want)[:, None, None] * nb).reshape(K, -1)
    k, i = torch.nonzero((at >= 0) & (at < nb), as_tuple=True)
    full = torch.zeros((K, nb + 2), dtype=torch.bool, device=c.device)
    full[:, 0] = full[:, -1] = True
    full[k, at[k, i].long() + 1] = True
    pos = torch.arange(nb + 2, device=c.device).expand(K, -1)
    last = torch.cummax(torch.where(full, pos, 0), dim=1).values
    gap = torch.where(full[:, 1:], pos[:, 1:] - last[:, :-1], 0)
    end = gap.argmax(dim=1)
    mid = end + 1 - gap.gather(1, end[:, None])[:, 0] / 2 - 0.5
    return (lo + 0.04 * want * mid / nb).float()


# ---------------------------------------------------------------- systems, kept as a program keeps them

_systems = {}


def _system(case):
    key = (case["rows"], case["cols"], case["scales"], case["batch"] if case.get("tuned") else 0)
    if key not in _systems:
        s = ShearletSystem.build(*key[:3])
        s.reserve(case["batch"])
        if case.get("tuned"):
            s.autotune(case["batch"])
        _systems[key] = s
    return _systems[key]


def _user_spectra(case):
    """A bank of 9 x 9 kernels (smaller where the image is) and one impulse, natural order, complex128 numpy."""
    rng = np.random.default_rng(case["rows"] * 7 + case["cols"] + case["filters"])
    ker = np.zeros((case["filters"], case["rows"], case["cols"]))
    r = np.arange(-4, 5)
    ker[:, (r % case["rows"])[:, None], (r % case["cols"])[None, :]] = rng.standard_normal((case["filters"], 9, 9)) / 9
    if case["real"]:
        ker = (ker + np.roll(ker[:, ::-1, ::-1], 1, axis=(1, 2))) / 2
    ker[-1] = 0
    ker[-1, 0, 0] = 1
    return np.fft.fft2(ker)


def _user_system(case):
    key = ("bank", case["rows"], case["cols"], case["filters"], case["real"])
    if key not in _systems:
        _systems[key] = ShearletSystem.from_spectra(np.fft.fftshift(_user_spectra(case), axes=(1, 2)))
    return _systems[key]


def _inpainter(case):
    if case["sizes"] not in _systems:
        _systems[case["sizes"]] = UnevenInpainter()
    return _systems[case["sizes"]]


# ---------------------------------------------------------------- denoising and inpainting inputs

_SIGMA = 30.0


def _denoise_thresholds(case, x):
    S = _bank(case["rows"], case["cols"], case["scales"])
    want = 3 * _SIGMA * _rms(S)
    return torch.stack([_in_gap(_sh(v[None], S)[0], want) for v in x])


def _inpaint_state(case, seed):
    """Masked images, masks and per-filter schedules: a geometric decay from the largest coefficient to 10 grey levels. Also the result in 64 bits."""
    its, images, masks, schedules, exact = case["iterations"], [], [], [], []
    for n, size in enumerate(int(v) for v in case["sizes"].split(",")):
        f = _images(size, size, 1, seed * 16 + n)[0]
        g = torch.Generator(device=DEV).manual_seed(seed * 16 + n + 1)
        mask = (torch.rand(f.shape, generator=g, device=DEV) < 0.5).float()
        fm = f * mask
        S = _bank(size, size, 3 if size <= 256 else 4)
        rms = _rms(S)
        first = float((_sh(fm[None], S)[0].abs().amax(dim=(1, 2)) / rms).max())
        u, rows = torch.zeros_like(f, dtype=torch.float64), []
        for i in range(its):
            c = _sh((mask * (fm - u) + u)[None], S)[0]
            rows.append(_in_gap(c, first * (10.0 / first) ** (i / max(1, its - 1)) * rms))
            u = _adj((c * (c.abs() >= rows[-1][:, None, None]))[None], S, True)[0]
        images.append(fm)
        masks.append(mask)
        schedules.append(torch.stack(rows).cpu().numpy())
        exact.append(u)
    return images, masks, schedules, exact


# ---------------------------------------------------------------- the shrinkage network's inputs

def _sigmas(case, seed):
    return torch.tensor(np.random.default_rng(seed).uniform(10, 50, case["batch"]).astype(np.float32), device=DEV)


def _params(K, seed):
    r = np.random.default_rng(seed)

    def he(co, ci):
        return (r.standard_normal((co, ci, 3, 3)) * np.sqrt(2 / (9 * ci))).astype(np.float32)

    p = {"W1": he(32, K), "b1": 0.1 * r.standard_normal(32), "W2": he(32, 32), "b2": 0.1 * r.standard_normal(32),
         "W3": 0.1 * he(K, 32), "b3": np.full(K, np.log(np.expm1(3.0)))}  # thresholds near 3 in noise units
    return {n: v.astype(np.float32) for n, v in p.items()}


def _moments(n, seed):
    """Adam's moments in mid-training."""
    r = np.random.default_rng(seed)
    return np.concatenate([1e-4 * r.standard_normal(n), 1e-6 * r.uniform(0.5, 2.0, n)]).astype(np.float32)


def _coefficients(case, seed, clean):
    """float32 coefficients of the noisy images (and of the clean ones), and the noise levels."""
    S, sg = _bank(case["rows"], case["cols"], case["scales"]), _sigmas(case, seed)
    size = (case["rows"], case["cols"], case["batch"], seed)
    noisy = torch.cat([_sh(v[None], S).float() for v in _images(*size, sg)])
    return noisy, torch.cat([_sh(v[None], S).float() for v in _images(*size)]) if clean else None, sg


_STEP, _LR, _TEMP = 500, 5e-4, 0.5


# ---------------------------------------------------------------- the interface

def prepare(case, seed):
    op = case["op"]
    if op == "inpaint":
        images, masks, schedules, _ = _inpaint_state(case, seed)
        return {"op": op, "inp": _inpainter(case), "images": images, "masks": masks, "schedules": schedules}
    if op == "bank":
        return {"op": op, "sys": _user_system(case), "x": _images(case["rows"], case["cols"], case["batch"], seed, 5.0)}
    system = _system(case)
    if op in ("apply", "train"):
        noisy, clean, sg = _coefficients(case, seed, op == "train")
        net = ShrinkNet(system, _params(system.K, seed))
        if op == "train":
            net.adam.copy_(torch.from_numpy(_moments(net.flat.numel(), seed)))
            net.steps = _STEP
        return {"op": op, "net": net, "c": noisy, "clean": clean, "sigma": sg, "tau": case.get("tau", False),
                "out": torch.empty_like(noisy) if op == "apply" else None}
    x = _images(case["rows"], case["cols"], case["batch"], seed, _SIGMA if op != "layer" else 0.0)
    if op == "layer":
        g = torch.randn((x.shape[0], system.K) + x.shape[1:], generator=torch.Generator(device=DEV).manual_seed(seed), device=DEV)
        return {"op": op, "layer": ShearletLayer(case["rows"], case["cols"], case["scales"], system=system),
                "x": x[:, None].clone().requires_grad_(True), "g": g}
    if op == "denoise":
        return {"op": op, "sys": system, "x": x, "thr": _denoise_thresholds(case, x), "y": torch.empty_like(x)}
    c = torch.empty((x.shape[0], system.K) + x.shape[1:], device=DEV)
    return {"op": op, "sys": system, "x": x, "c": c, "y": torch.empty_like(x)}


def run(s):
    op = s["op"]
    if op == "fwdinv":
        s["sys"].forward(s["x"], out=s["c"])
        s["sys"].inverse(s["c"], out=s["y"])
        return s["c"], s["y"]
    if op == "bank":
        c = s["sys"].forward(s["x"])
        return c, s["sys"].inverse(c)
    if op == "layer":
        s["x"].grad = None
        c = s["layer"](s["x"])
        c.backward(s["g"])
        return c, s["x"].grad
    if op == "denoise":
        return s["sys"].denoise(s["x"], s["thr"], out=s["y"], kept=True)
    if op == "inpaint":
        return s["inp"].run(s["images"], s["masks"], s["schedules"])
    if op == "apply":
        return s["net"].apply(s["c"], s["sigma"], out=s["out"], tau=s["tau"])
    loss = s["net"].train_step(s["c"], s["clean"], s["sigma"], lr=_LR, temperature=_TEMP)
    return loss, s["net"].grads, s["net"].flat


def work(case):
    """Inputs read once, outputs written once (filter sets included); 2.5 n log2 n operations for a real FFT of n points."""
    op = case["op"]

    def transform(rows, cols, k, b, directions, per_value=4):
        n = rows * cols
        return directions * (per_value * k * rows * (cols // 2 + 1)), directions * b * ((k + 1) * 2.5 * n * math.log2(n) + k * 3 * n)

    if op == "inpaint":
        by = fl = 0.0
        sizes = [int(v) for v in case["sizes"].split(",")]
        for n in sorted(set(sizes)):
            b, f = transform(n, n, _filters(3 if n <= 256 else 4), sizes.count(n), 2)
            by += case["iterations"] * (b + sizes.count(n) * 16 * n * n)
            fl += case["iterations"] * f
        return {"bytes": by, "flops": fl}
    rows, cols, B = case["rows"], case["cols"], case["batch"]
    K = case["filters"] if op == "bank" else _filters(case["scales"])
    pix = B * rows * cols
    if op in ("apply", "train"):
        flops = 2 * 9 * 32 * pix * (2 * K + 32)
        if op == "train":
            return {"bytes": 8.0 * K * pix, "flops": 3.0 * flops}
        return {"bytes": (12.0 if case["tau"] else 8.0) * K * pix, "flops": flops}
    by, fl = transform(rows, cols, K, B, 2, 8 if op == "bank" and not case["real"] else 4)
    return {"bytes": by + 8.0 * pix + (0.0 if op == "denoise" else 8.0 * K * pix), "flops": fl}


# ---------------------------------------------------------------- the results in 64 bits

def _taps(x):
    """(9 C, pixels): the nine circular neighbours of every pixel of x (C, rows, cols), tap-major."""
    return torch.stack([torch.roll(x, (1 - dy, 1 - dx), (1, 2)) for dy in range(3) for dx in range(3)]).reshape(9 * x.shape[0], -1)


def _mat(W):
    return W.permute(0, 2, 3, 1).reshape(W.shape[0], -1)


def _conv(x, W, b=0.0):
    return (_mat(W) @ _taps(x)).reshape(W.shape[0], *x.shape[1:]) + b


def _network(case, seed, c, clean, sg):
    """Thresholds in noise units of the images; with `clean`, the training loss and the gradients, flat. Operands are rounded to bfloat16 where the network's are."""
    def r(v):
        return v.float().bfloat16().double()

    p = {n: torch.from_numpy(v).to(DEV).double() for n, v in _params(c.shape[1], seed).items()}
    W1, W2, W3 = r(p["W1"]), r(p["W2"]), r(p["W3"])
    b1, b2, b3 = (p[n][:, None, None] for n in ("b1", "b2", "b3"))
    K, taus, loss, grads = c.shape[1], [], 0.0, {n: torch.zeros_like(v) for n, v in p.items()}
    rms = _rms(_bank(case["rows"], case["cols"], case["scales"]))
    weight = 1.0 / (c.shape[0] * (K - 1) * c.shape[2] * c.shape[3])

    def wgrad(d, x):
        return (d.reshape(d.shape[0], -1) @ _taps(x).T).reshape(d.shape[0], 3, 3, x.shape[0]).permute(0, 3, 1, 2)

    def back(d, W):
        return _conv(d, W.flip(2, 3).transpose(0, 1))

    for v, w, s in zip(c, clean if clean is not None else c, sg.double()):
        scale = 1 / (s * rms)[:, None, None]
        z = v.double() * scale
        zb = r(z)
        h1 = r(_conv(zb, W1, b1).relu())
        h2 = r(_conv(h1, W2, b2).relu())
        o = _conv(h2, W3, b3)
        tau = torch.nn.functional.softplus(o, threshold=100.0)
        tau[-1] = 0
        if clean is None:
            taus.append(tau)
            continue
        g = torch.sigmoid((z.abs() - tau) / _TEMP)
        res = (z * g - w.double() * scale)[:-1]
        loss = loss + weight * res.square().sum()
        do = torch.zeros_like(z)
        do[:-1] = r(-2 * weight / _TEMP * res * (z * g * (1 - g) * torch.sigmoid(o))[:-1])
        dh2 = r(back(do, W3) * (h2 > 0))
        dh1 = r(back(dh2, W2) * (h1 > 0))
        for n, d, x in (("3", do, h2), ("2", dh2, h1), ("1", dh1, zb)):
            grads["W" + n] += wgrad(d, x)
            grads["b" + n] += d.sum(dim=(1, 2))
    if clean is None:
        return torch.stack(taus)
    names = ("W1", "b1", "W2", "b2", "W3", "b3")
    return loss.reshape(1), torch.cat([grads[n].reshape(-1) for n in names]), torch.cat([p[n].reshape(-1) for n in names])


def exact(case, seed):
    op = case["op"]
    if op == "inpaint":
        return _inpaint_state(case, seed)[3]
    if op == "bank":
        S = torch.from_numpy(_user_spectra(case)).to(DEV)
        x = _images(case["rows"], case["cols"], case["batch"], seed, 5.0)
        return _sh(x, S), x.double()
    S = _bank(case["rows"], case["cols"], case["scales"])
    if op in ("apply", "train"):
        c, clean, sg = _coefficients(case, seed, op == "train")
        if op == "apply":
            tau = _network(case, seed, c, None, sg)
            keep = (c.double() / (sg.double()[:, None] * _rms(S))[:, :, None, None]).abs() >= tau
            return (c.double() * keep, tau) if case["tau"] else c.double() * keep
        loss, g, p = _network(case, seed, c, clean, sg)
        m, v = torch.from_numpy(_moments(g.numel(), seed)).to(DEV).double().chunk(2)
        m, v = 0.9 * m + 0.1 * g, 0.999 * v + 0.001 * g * g
        t = _STEP + 1
        return loss, g, p - _LR * (m / (1 - 0.9 ** t)) / ((v / (1 - 0.999 ** t)).sqrt() + 1e-8)
    x = _images(case["rows"], case["cols"], case["batch"], seed, _SIGMA if op != "layer" else 0.0)
    if op == "layer":
        g = torch.randn((x.shape[0], S.shape[0]) + x.shape[1:], generator=torch.Generator(device=DEV).manual_seed(seed), device=DEV)
        return _sh(x, S), _adj(g, S, False)[:, None]
    if op == "denoise":
        keep = [(c, c.abs() >= t[:, None, None]) for c, t in zip(_sh(x, S), _denoise_thresholds(case, x))]
        return torch.cat([_adj((c * k)[None], S, True) for c, k in keep]), torch.stack([k.sum(dim=(1, 2)) for _, k in keep])
    return _sh(x, S), x.double()

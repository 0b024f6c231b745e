"""What the framework's speed is measured on: the calls that a user's program makes through
`paper_2106_12736_amd.layers`, over the sizes that such programs have.

The paper trains an FDCNN on grayscale fundus photographs of 512 x 512, 4 images a step; the
benchmark's stacks take 256 x 256 to 1024 x 1024 images, 8 to 32 a step; its Full FDC layers are
convolution layers of a VGG16 on 224 x 224 and 512 x 512 images.  The paths, each through the class
or functions that a program uses:

  layer          CicLayer: one CIC + FDP layer with spectral kernels, forward and backward
  spatial        CicSpatialLayer: the same with n x n spatial kernels (with M = N, the CIC form of a
                 VGG16's convolution layer)
  stack          CicStackFused: a CIC + FDP network body, a training step or inference alone
  spatial_stack  CicSpatialStackFused: the same body with n x n spatial kernels
  classifier     FdcnnClassifier: a whole training step (spectral chain, head, loss, Adam)
  spectral       the separate operations (FftPlan, cic_*, fdp_*), composed by the caller
  full           FullLayer: a Full FDC layer (contraction over input channels), forward and backward

Everything is float32 / complex64, as the framework is.
"""

import math

import torch

from paper_2106_12736_amd import layers

DEV = "cuda"


# ----------------------------------------------------------------------------
# cases
# ----------------------------------------------------------------------------
def listed():
    return [
        # a first small layer of 2 images: the least work a call can be given, launches and latency
        {"name": "layer_64_b2", "path": "layer", "B": 2, "C": 1, "S": 4, "N": 64, "M": 32, "artifact": "none", "n": 1},
        # a first layer on colour images, an odd batch, 8 kernels a channel, the artifact rows cut off
        {"name": "layer_256_rgb_b5", "path": "layer", "B": 5, "C": 3, "S": 24, "N": 256, "M": 128,
         "artifact": "crop", "n": 5},
        # Conv Block 4 of a VGG16 on 512 x 512 images with CIC in place of its convolution
        {"name": "spatial_64_c256_512_b16", "path": "spatial", "B": 16, "C": 256, "S": 512, "N": 64, "M": 64,
         "artifact": "crop", "n": 3},
        # training steps of a small and of the largest network body
        {"name": "stack_256_b16", "path": "stack", "B": 16, "C": 1, "width": 8, "N": 256, "M": 32, "train": True},
        {"name": "stack_1024_b8", "path": "stack", "B": 8, "C": 1, "width": 8, "N": 1024, "M": 32, "train": True},
        # one large photograph through the trained body
        {"name": "stack_1024_b1_infer", "path": "stack", "B": 1, "C": 1, "width": 8, "N": 1024, "M": 32,
         "train": False},
        # the paper's image size and batch with kernels that are small and spatial, as section 2.4.1.2 has them
        {"name": "spatial_stack_512_b4", "path": "spatial_stack", "B": 4, "C": 1, "width": 8, "N": 512, "M": 32,
         "n": 3},
        # the paper's training step at its image size and batch
        {"name": "classifier_512_b4", "path": "classifier", "B": 4, "C": 1, "width": 8, "N": 512, "M": 32},
        # a layer composed of the separate operations at the sizes of the paper's layer timings
        {"name": "spectral_512_b4", "path": "spectral", "B": 4, "C": 8, "S": 16, "N": 512, "M": 256},
        # convolution layers as Full FDC: the benchmark's batch, the paper's batch, and sizes that fill no tile
        {"name": "full_224_c64_b16", "path": "full", "B": 16, "C": 64, "S": 64, "N": 224, "artifact": "crop", "n": 3},
        {"name": "full_512_c128_b4", "path": "full", "B": 4, "C": 128, "S": 128, "N": 512, "artifact": "crop", "n": 3},
        {"name": "full_128_c48_80_b3", "path": "full", "B": 3, "C": 48, "S": 80, "N": 128, "artifact": "roll", "n": 5},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_once(rng):
    path = rng.choice(["layer", "spatial", "stack", "stack", "spatial_stack", "classifier", "spectral", "full",
                       "full", "full"])
    if path in ("stack", "spatial_stack", "classifier"):
        C = rng.choice([1, 1, 1, 3])  # grayscale, as in the paper, or colour
        c = {"path": path, "B": _log_int(rng, 1, 32), "C": C, "width": C * rng.choice([4, 6, 8]) if C == 3 else
             rng.choice([4, 8, 8, 16]), "N": rng.choice([128, 256, 512, 1024]), "M": rng.choice([32, 32, 16])}
        if path == "stack":
            c["train"] = rng.random() < 0.6
        if path == "spatial_stack":
            c["n"] = rng.choice([3, 3, 5, 7])
        return c
    if path in ("layer", "spatial"):
        C = rng.choice([1, 3, _log_int(rng, 4, 256)])
        N = rng.choice([32, 64, 128, 256, 512, 1024])
        M = N if path == "spatial" and rng.random() < 0.5 else N // rng.choice([2, 2, 4])
        return {"path": path, "B": _log_int(rng, 1, 32), "C": C, "S": C * rng.choice([1, 2, 2, 4, 5, 8]), "N": N,
                "M": M, "artifact": rng.choice(["none", "crop", "roll"]), "n": rng.choice([1, 3, 5, 7])}
    if path == "spectral":
        C = _log_int(rng, 1, 64)
        N = rng.choice([32, 64, 128, 224, 256, 512, 1024])
        return {"path": path, "B": _log_int(rng, 1, 32), "C": C, "S": C * rng.choice([1, 2, 2, 4]), "N": N,
                "M": N // 2 if N != 224 else 128}
    return {"path": path, "B": _log_int(rng, 1, 20), "C": _log_int(rng, 3, 256), "S": _log_int(rng, 16, 512),
            "N": rng.choice([32, 64, 128, 224, 224, 256, 512]), "artifact": rng.choice(["crop", "crop", "roll"]),
            "n": rng.choice([3, 3, 3, 5])}


def _cost(case):
    """A rough count of a pass's work, to keep drawn cases within the listed ones."""
    B, C, N = case["B"], case["C"], case["N"]
    if case["path"] == "full":
        S = case["S"]
        return 8 * N * N * (B * C + B * S) * 6 + 12 * (B + 3) * C * S * N * N / 20
    if "width" in case:
        total, w = 0, case["width"]
        while N > case["M"]:
            total += 8 * N * N * (B * C + B * w + w) * 2
            C, w, N = w, 2 * w, N // 2
        return total
    return 8 * N * N * (B * C + B * case["S"] + case["S"]) * 4


def draw(rng):
    most = max(_cost(c) for c in listed())
    while True:
        c = _draw_once(rng)
        if 1e5 <= _cost(c) <= most and c.get("n", 1) <= c.get("M", c["N"]):
            return c


def _geometry(case):
    """Sizes and channels of every layer of a body: halving from N to M, the channels doubling after the first."""
    sizes, channels = [case["N"]], [case["C"]]
    while sizes[-1] > case["M"]:
        sizes.append(sizes[-1] // 2)
        channels.append(case["width"] if len(channels) == 1 else 2 * channels[-1])
    return sizes, channels


def _out(case):
    M = case.get("M", case["N"])
    return M - case["n"] + 1 if case["artifact"] == "crop" else M


# ----------------------------------------------------------------------------
# inputs and the pass
# ----------------------------------------------------------------------------
def _images(g, B, C, N):
    """Fundus-like images in [0, 1]: a textured disc with a vignette on black."""
    t = (torch.arange(N, device=DEV) + 0.5) * (2.0 / N) - 1.0
    r = torch.sqrt(t[:, None] ** 2 + t[None, :] ** 2)
    disc = torch.sigmoid((0.92 - r) / 0.015) * (1.0 - 0.4 * r * r)
    return torch.rand((B, C, N, N), generator=g, device=DEV) * disc


def _spectra(g, S, N):
    return torch.view_as_complex(torch.randn((S, N, N // 2 + 1, 2), generator=g, device=DEV) * 0.1)


def _tensors(case, seed):
    """The inputs of a case, from the seed alone."""
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    path, B, C, N = case["path"], case["B"], case["C"], case["N"]

    def normal(*shape, std=1.0):
        return torch.randn(shape, generator=g, device=DEV) * std

    if path in ("stack", "spatial_stack", "classifier"):
        sizes, channels = _geometry(case)
        x = _images(g, B, C, N)
        if path == "spatial_stack":
            n = case["n"]
            k = [normal(s, n, n, std=math.sqrt(2.0) / n) for s in channels[1:]]
        else:
            k = [_spectra(g, s, N) for s, N in zip(channels[1:], sizes)]
        if path == "classifier":
            F = channels[-1] * sizes[-1] ** 2
            return x, k, normal(2, F, std=math.sqrt(2.0 / F)), normal(2, std=0.01), \
                torch.randint(0, 2, (B,), generator=g, device=DEV, dtype=torch.int32)
        return x, k, normal(B, channels[-1], sizes[-1], sizes[-1])
    S = case["S"]
    if path == "spectral":
        return normal(B, C, N, N), _spectra(g, S, N), normal(B, S, case["M"], case["M"])
    x = _images(g, B, C, N) if path == "layer" and C in (1, 3) else normal(B, C, N, N)
    n = case["n"]
    if path == "layer":
        k = _spectra(g, S, N)
    elif path == "spatial":
        k = normal(S, n, n, std=math.sqrt(2.0) / n)
    else:
        k = normal(S, C, n, n, std=math.sqrt(2.0 / C) / n)
    return x, k, normal(B, S, _out(case), _out(case))


def prepare(case, seed):
    path, B, C, N = case["path"], case["B"], case["C"], case["N"]
    st = {"path": path, "t": _tensors(case, seed), "train": case.get("train", True)}
    if path in ("stack", "spatial_stack", "classifier"):
        sizes, channels = _geometry(case)
        if path == "stack":
            st["m"] = layers.CicStackFused(B, sizes, channels)
        elif path == "spatial_stack":
            st["m"] = layers.CicSpatialStackFused(B, sizes, channels, case["n"])
        else:
            st["m"] = layers.FdcnnClassifier(B, sizes, channels)
            st["m"].load(*st["t"][1:4])
        return st
    S, M = case["S"], case.get("M", N)
    if path == "layer":
        st["m"] = layers.CicLayer(B, C, S, N, M, artifact=case["artifact"], kernel_n=case["n"])
    elif path == "spatial":
        st["m"] = layers.CicSpatialLayer(B, C, S, N, M, case["n"], artifact=case["artifact"])
    elif path == "full":
        st["m"] = layers.FullLayer(B, C, S, N, kernel_n=case["n"], artifact=case["artifact"])
    else:
        st["m"] = layers.FftPlan(B * C, N, N), layers.FftPlan(B * S, M, M)
        return st
    st["saved"] = st["m"].new_saved()
    return st


def run(st):
    path, m = st["path"], st["m"]
    if path in ("stack", "spatial_stack"):
        x, k, gy = st["t"]
        y = m.forward(x, k)
        return {"y": y, "gk": m.backward(gy, k)} if st["train"] else {"y": y}
    if path == "classifier":
        x, _, _, _, labels = st["t"]
        loss = m.train_step(x, labels)
        return {"loss": loss, "logits": m.logits, "grads": m.grads, "params": m.params, "m": m.m, "v": m.v}
    x, k, gy = st["t"]
    if path == "spectral":
        fine, coarse = m
        N, M = fine.h, coarse.h
        X = fine.rfft2(x)
        y = coarse.irfft2(layers.fdp_forward(layers.cic_forward(X, k), M, M))
        gX, gk = layers.cic_backward(layers.fdp_backward(coarse.irfft2_backward(gy), N, N), X, k)
        return {"y": y, "gx": fine.rfft2_backward(gX), "gk": gk}
    y = m.forward(x, k, saved=st["saved"])
    gx, gk = m.backward(gy, st["saved"], k)
    return {"y": y, "gx": gx, "gk": gk}


# ----------------------------------------------------------------------------
# work and tolerance
# ----------------------------------------------------------------------------
def _fft2(planes, n, kept=None):
    """Operations of `planes` real 2-D transforms of n x n of which kept x (kept/2+1) bins are needed:
    2.5 n log2 n a real row, 5 n log2 n a kept column."""
    kept = n if kept is None else kept
    return planes * (n * 2.5 * n + (kept // 2 + 1) * 5.0 * n) * math.log2(n)


def work(case):
    path, B, C, N = case["path"], case["B"], case["C"], case["N"]
    passes = 2 if case.get("train", True) else 1  # forward, and backward
    if path in ("stack", "spatial_stack", "classifier"):
        sizes, channels = _geometry(case)
        flops = kbytes = kfull = 0
        for i, s in enumerate(channels[1:]):
            n, m = sizes[i], sizes[i + 1]
            bins = m * (m // 2 + 1)
            kbytes += 8 * s * bins
            kfull += 8 * s * n * (n // 2 + 1)
            flops += (8 * B * s * bins) * (1 if passes == 1 else 3 if i else 2)
            if path != "classifier":
                flops += passes * _fft2(B * s, m) + (passes if i else 1) * _fft2(B * channels[i], n, m)
        if path == "classifier":
            flops += _fft2(B * C, N, sizes[1]) + 2 * _fft2(B * channels[-1], sizes[-1])
        out = 4 * B * channels[-1] * sizes[-1] ** 2
        nbytes = 4 * B * C * N * N + out
        if path == "classifier":
            params = kfull + 4 * 2 * (channels[-1] * sizes[-1] ** 2 + 1)
            return {"bytes": nbytes - out + 6 * params + kbytes, "flops": flops + 3.0 * params}  # Adam's p, m, v
        if path == "spatial_stack":
            return {"bytes": nbytes + out + 2 * 4 * sum(channels[1:]) * case["n"] ** 2, "flops": flops}
        return {"bytes": nbytes + kbytes + (out + kbytes if passes == 2 else 0), "flops": flops}
    S, M = case["S"], case.get("M", N)
    o = M if path == "spectral" else _out(case)
    nbytes = 2 * 4 * (B * C * N * N + B * S * o * o)  # x, gx, y, gy
    bins = M * (M // 2 + 1)
    flops = 2 * (_fft2(B * C, N, M) + _fft2(B * S, M))
    if path == "full":
        return {"bytes": nbytes + 2 * 4 * S * C * case["n"] ** 2, "flops": flops + 3 * 8.0 * B * S * C * bins}
    flops += 3 * 8.0 * B * S * bins
    if path == "spatial":
        return {"bytes": nbytes + 2 * 4 * S * case["n"] ** 2, "flops": flops}
    return {"bytes": nbytes + 8 * S * (bins + N * (N // 2 + 1)), "flops": flops}


def tolerance(case):
    # About four times the error of float32 against float64 that these paths show (up to 6e-7
    # for a body of five layers, each four transforms and a product).
    if case["path"] == "classifier":
        # a feature within rounding of 0 may pass the ReLU on one side only, which moves the
        # gradient of one feature of B * F / 2 by its whole size
        return {"rel": 5e-3, "max": 0.5}
    return {"rel": 2.5e-6, "max": 1e-4}


# ----------------------------------------------------------------------------
# the same in 64 bits
# ----------------------------------------------------------------------------
def _rfft2(x):
    return torch.fft.rfft2(x)


def _irfft2(Y):
    """The inverse with real-part semantics: after the column inverse, the imaginary parts of
    columns 0 and W/2 are dropped."""
    Z = torch.fft.ifft(Y, dim=-2)
    real = torch.complex(Z.real, torch.zeros_like(Z.real))
    Z = torch.cat([real[..., :1], Z[..., 1:-1], real[..., -1:]], dim=-1)
    return torch.fft.irfft(Z, n=2 * (Z.shape[-1] - 1), dim=-1)


def _fdp(X, M):
    N = X.shape[-2]
    return torch.cat([X[..., : M // 2, : M // 2 + 1], X[..., N - M // 2:, : M // 2 + 1]], dim=-2)


def _cic(X, K):
    return X.repeat_interleave(K.shape[0] // X.shape[1], dim=1) * K


def _artifact(y, artifact, n):
    if artifact == "crop":
        return y[..., n - 1:, n - 1:]
    if artifact == "roll":
        s = (n - 1) // 2
        return torch.roll(y, (-s, -s), (-2, -1))
    return y


def _pad(w, N):
    return torch.nn.functional.pad(w, (0, N - w.shape[-1], 0, N - w.shape[-2]))


def _wide(t):
    return t.to(torch.complex128 if t.is_complex() else torch.float64)


def exact(case, seed):
    t = _tensors(case, seed)
    path = case["path"]
    if path == "full":
        return _exact_full(case, *(_wide(v) for v in t))
    x = _wide(t[0])
    several = isinstance(t[1], list)
    ks = [_wide(k).requires_grad_() for k in (t[1] if several else [t[1]])]
    if path == "classifier":
        return _exact_classifier(case, x, ks, _wide(t[2]), _wide(t[3]), t[4].long())
    train = case.get("train", True)
    if not several:
        x.requires_grad_()
    with torch.set_grad_enabled(train):
        if several:
            sizes, _ = _geometry(case)
            h = x
            for k, M in zip(ks, sizes[1:]):
                h = _layer(h, k, M, "roll" if path == "spatial_stack" else "none", case.get("n", 1))
        else:
            h = _layer(x, ks[0], case["M"], case.get("artifact", "none"), case.get("n", 1))
    if not train:
        return {"y": h}
    h.backward(_wide(t[2]))
    gk = [k.grad for k in ks]
    if several:
        return {"y": h.detach(), "gk": gk}
    return {"y": h.detach(), "gx": x.grad, "gk": gk[0]}


def _layer(x, k, M, artifact, n):
    """One layer; k complex spectra, or real n x n kernels."""
    if not k.is_complex():
        k = _rfft2(_pad(k, x.shape[-1]))
    return _artifact(_irfft2(_cic(_fdp(_rfft2(x), M), _fdp(k, M))), artifact, n)


def _exact_classifier(case, x, ks, W, bias, labels):
    sizes, _ = _geometry(case)
    W.requires_grad_()
    bias.requires_grad_()
    Z = _rfft2(x)
    for k, M in zip(ks, sizes[1:]):
        Z = _cic(_fdp(Z, M), _fdp(k, M))
    logits = torch.relu(_irfft2(Z)).flatten(1) @ W.T + bias
    loss = torch.nn.functional.cross_entropy(logits, labels)
    loss.backward()

    def flat(ts):
        return torch.cat([(torch.view_as_real(v) if v.is_complex() else v).reshape(-1) for v in ts])

    with torch.no_grad():
        p, g = flat(ks + [W, bias]), flat([v.grad for v in ks + [W, bias]])
        wg = g + 1e-6 * p
        m, v = 0.1 * wg, 0.001 * wg * wg
        p = p - 1e-5 * (m / 0.1) / (torch.sqrt(v / 0.001) + 1e-8)
        return {"loss": loss.detach().reshape(1), "logits": logits.detach(), "grads": g, "params": p, "m": m, "v": v}


def _exact_full(case, x, w, gy):
    """The circular convolution over the input channels, tap by tap, and its adjoints."""
    B, C, N, _ = x.shape
    S, n = w.shape[0], w.shape[-1]
    if case["artifact"] == "crop":
        g = torch.nn.functional.pad(gy, (n - 1, 0, n - 1, 0))
    else:
        s = (n - 1) // 2
        g = torch.roll(gy, (s, s), (-2, -1))
    g = g.reshape(B, S, N * N)
    y, gx, gw = torch.zeros_like(g), torch.zeros_like(x), torch.zeros_like(w)
    for a in range(n):
        for b in range(n):
            xs = torch.roll(x, (a, b), (-2, -1)).reshape(B, C, N * N)
            for i in range(B):
                y[i].addmm_(w[:, :, a, b], xs[i])
                gw[:, :, a, b] += g[i] @ xs[i].T.contiguous()
                gx[i] += torch.roll((w[:, :, a, b].T.contiguous() @ g[i]).reshape(C, N, N), (-a, -b), (-2, -1))
    return {"y": _artifact(y.reshape(B, S, N, N), case["artifact"], n), "gx": gx, "gk": gw}

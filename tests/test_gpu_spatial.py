"""GPU parity of the CIC + FDP layer with spatial n x n kernels (kernel spectra formed
on every call, section 2.4.1.2) and its weight gradient, against the float64 oracle:
single layers over sizes, poolings, kernel sizes and artifact modes, and a full-size
stack in the configuration the benchmark times with --spatial-kernel 3."""

import zlib

import numpy as np
import pytest
import torch

from _parity import assert_parity, to_np
from oracle import fdc
from paper_2106_12736_amd import inputs, layers

pytestmark = pytest.mark.gpu

MODE = {"none": fdc.ARTIFACT_NONE, "crop": fdc.ARTIFACT_CROP, "roll": fdc.ARTIFACT_ROLL}


def _rng(*key):
    return np.random.default_rng(zlib.crc32(repr(key).encode()))


CASES = [
    # N, M, B, C, J, n, artifact
    (16, 16, 2, 1, 3, 3, "crop"),
    (16, 8, 2, 2, 2, 3, "roll"),
    (32, 16, 1, 1, 4, 5, "crop"),
    (64, 32, 2, 1, 4, 1, "none"),
    (64, 64, 1, 2, 2, 8, "roll"),
    (128, 64, 2, 1, 2, 3, "crop"),
    (224, 224, 1, 1, 2, 3, "roll"),
    (512, 256, 1, 1, 2, 5, "crop"),
    (1024, 512, 1, 1, 2, 3, "roll"),
]


@pytest.mark.parametrize("N,M,B,C,J,n,artifact", CASES)
def test_spatial_layer(N, M, B, C, J, n, artifact):
    print(f"spatial N={N} M={M} B={B} C={C} J={J} n={n} {artifact}", flush=True)
    rng = _rng("spatial", N, M, B, C, J, n, artifact)
    S = C * J
    x = inputs.normal(rng, (B, C, N, N))
    w = inputs.normal(rng, (S, n, n)) * np.float32(np.sqrt(2.0 / (n * n)))
    layer = layers.CicSpatialLayer(B, C, S, N, M, n, artifact=artifact)
    gy = inputs.normal(rng, (B, S, layer.out, layer.out))
    xd, wd = torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda()
    saved = layer.new_saved()
    y = layer.forward(xd, wd, saved=saved)
    gx, gw = layer.backward(torch.from_numpy(gy).cuda(), saved, wd)
    torch.cuda.synchronize()
    y_ref, xs = fdc.cic_spatial_layer_forward(x.astype(np.float64), w.astype(np.float64), M, MODE[artifact])
    gx_ref, gw_ref = fdc.cic_spatial_layer_backward(gy.astype(np.float64), xs, w.astype(np.float64), M,
                                                    MODE[artifact])
    assert_parity(to_np(y), y_ref, "y")
    assert_parity(to_np(gx), gx_ref, "gx")
    assert_parity(to_np(gw), gw_ref, "gw")


@pytest.mark.parametrize("wl", [inputs.STACK256, inputs.STACK1024], ids=lambda w: w.name)
def test_spatial_stack(wl):
    print(f"spatial stack {wl.name}", flush=True)
    n = 3
    d = inputs.make_cic_spatial(wl, n)
    st = layers.CicSpatialStack(wl.batch, wl.sizes, wl.channels, n)
    x = torch.from_numpy(d.x).cuda()
    ws = [torch.from_numpy(w).cuda() for w in d.weights]
    gin = torch.empty_like(x)
    st.forward(x, ws)
    st.backward(torch.from_numpy(d.grad).cuda(), ws, input_grad=gin)
    torch.cuda.synchronize()
    h = d.x.astype(np.float64)
    saved = []
    for i in range(wl.layers):
        h, xs = fdc.cic_spatial_layer_forward(h, d.weights[i].astype(np.float64), wl.sizes[i + 1], fdc.ARTIFACT_ROLL)
        saved.append(xs)
    assert_parity(to_np(st.acts[-1]), h, "y")
    g = d.grad.astype(np.float64)
    for i in reversed(range(wl.layers)):
        g, gw = fdc.cic_spatial_layer_backward(g, saved[i], d.weights[i].astype(np.float64), wl.sizes[i + 1],
                                               fdc.ARTIFACT_ROLL)
        assert_parity(to_np(st.gws[i]), gw, f"gw[{i}]")
    assert_parity(to_np(gin), g, "gx")


def _oracle_roll_stack(x, weights, sizes, grad):
    """The spatial stack layer after layer with ROLL (the oracle's layer functions)."""
    h, saved = x.astype(np.float64), []
    for i, w in enumerate(weights):
        h, xs = fdc.cic_spatial_layer_forward(h, w.astype(np.float64), sizes[i + 1], fdc.ARTIFACT_ROLL)
        saved.append(xs)
    g, gws = grad.astype(np.float64), [None] * len(weights)
    for i in reversed(range(len(weights))):
        g, gws[i] = fdc.cic_spatial_layer_backward(g, saved[i], weights[i].astype(np.float64), sizes[i + 1],
                                                   fdc.ARTIFACT_ROLL)
    return h, gws, g


FUSED_SPATIAL = [
    # workload (or batch, sizes, channels), n: ROLL shifts 0 .. 3
    (inputs.LAYER64, 5), (inputs.STACK256, 3), (inputs.STACK512, 2), (inputs.STACK1024, 3),
    ((3, (64, 32, 16), (2, 4, 8)), 4), ((2, (32, 16), (1, 3)), 7), ((2, (16, 16, 8), (1, 2, 2)), 1),
]


@pytest.mark.parametrize("case,n", FUSED_SPATIAL, ids=lambda v: getattr(v, "name", str(v)))
def test_spatial_stack_fused(case, n):
    """fdc_cic_spatial_stack_*: every layer's kernel spectra with the ROLL phase in one
    launch, the stack executor, every dL/dw in one launch; against the oracle's layers."""
    if isinstance(case, inputs.CicStack):
        d = inputs.make_cic_spatial(case, n)
        B, sizes, chans = case.batch, case.sizes, case.channels
        x, weights, grad = d.x, d.weights, d.grad
    else:
        B, sizes, chans = case
        rng = _rng("spatial_fused", B, sizes, chans, n)
        x = inputs.normal(rng, (B, chans[0], sizes[0], sizes[0]))
        weights = [inputs.normal(rng, (chans[i + 1], n, n)) * np.float32(np.sqrt(2.0 / (n * n)))
                   for i in range(len(sizes) - 1)]
        grad = inputs.normal(rng, (B, chans[-1], sizes[-1], sizes[-1]))
    print(f"spatial stack fused {sizes} {chans} B={B} n={n}", flush=True)
    st = layers.CicSpatialStackFused(B, sizes, chans, n)
    xd = torch.from_numpy(x).cuda()
    ws = [torch.from_numpy(w).cuda() for w in weights]
    gin = torch.empty_like(xd)
    y = st.forward(xd, ws).clone()
    gws = [g.clone() for g in st.backward(torch.from_numpy(grad).cuda(), ws, input_grad=gin)]
    torch.cuda.synchronize()
    y_ref, gw_ref, gx_ref = _oracle_roll_stack(x, weights, sizes, grad)
    assert_parity(to_np(y), y_ref, "y")
    for i in range(len(weights)):
        assert_parity(to_np(gws[i]), gw_ref[i], f"gw[{i}]")
    assert_parity(to_np(gin), gx_ref, "gx")
    # a second call on the same buffers gives identical results (fixed summation order)
    st.forward(xd, ws)
    again = st.backward(torch.from_numpy(grad).cuda(), ws, input_grad=gin)
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(gws, again))


@pytest.mark.parametrize("wl", inputs.FULL_CIC_WORKLOADS, ids=lambda w: w.name)
def test_full_fdc_with_cic_block4(wl):
    """The Full FDC layer with CIC at the paper's VGG16 Conv Block 4 shapes (64 x 64,
    256 -> 512 and 512 -> 512 channels, 3 x 3, crop), 16 images, in the configuration
    the benchmark times; every output element against the oracle."""
    print(f"full cic {wl.name}", flush=True)
    d = inputs.make_full_cic(wl)
    layer = layers.CicSpatialLayer(wl.batch, wl.cin, wl.cout, wl.size, wl.size, wl.n, artifact="crop")
    xd, wd = torch.from_numpy(d.x).cuda(), torch.from_numpy(d.w).cuda()
    saved = layer.new_saved()
    y = layer.forward(xd, wd, saved=saved)
    gx, gw = layer.backward(torch.from_numpy(d.grad).cuda(), saved, wd)
    torch.cuda.synchronize()
    y_ref, xs = fdc.cic_spatial_layer_forward(d.x.astype(np.float64), d.w.astype(np.float64), wl.size,
                                              fdc.ARTIFACT_CROP)
    gx_ref, gw_ref = fdc.cic_spatial_layer_backward(d.grad.astype(np.float64), xs, d.w.astype(np.float64), wl.size,
                                                    fdc.ARTIFACT_CROP)
    assert_parity(to_np(y), y_ref, "y")
    assert_parity(to_np(gx), gx_ref, "gx")
    assert_parity(to_np(gw), gw_ref, "gw")


# Partials of dL/dw per output channel: 2, 8 x 5 and 8 x 5
@pytest.mark.parametrize("N,M,C,J,n", [(64, 64, 16, 4, 3), (512, 512, 4, 4, 5), (1024, 512, 4, 4, 3)])
def test_spatial_weight_gradient_rounding(N, M, C, J, n):
    """dL/dw's sums over the kept bins of dK, against the same dK summed in 64 bits.  In units of
    a rounding's rms, u = 2.5e-8, and with terms of random signs, m additions in a row add m u^2 / 2 to
    the square of the error: 4 for the 8 multiply-adds of four rows, 2 for four such sums, 2 for the
    projection, 8 for the levels of 256 lanes (a tree adds u^2 a level) and 1 for the twiddles; the sum over
    workgroups is in 64 bits.  4.1 u = 1.03e-7, and 1.18e-7 leaves 15 %.  All 16 rows in one chain would be
    1.3e-7, 40 workgroups added in 32 bits 1.7e-7."""
    rng = _rng("spatial wgrad", N, M, C, J, n)
    S = C * J
    x, w = inputs.normal(rng, (1, C, N, N)), inputs.normal(rng, (S, n, n))
    spatial = layers.CicSpatialLayer(1, C, S, N, M, n, artifact="crop")
    layer = layers.CicLayer(1, C, S, N, M, "crop", n)
    xd, wd = torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda()
    gy = torch.from_numpy(inputs.normal(rng, (1, S, layer.out, layer.out))).cuda()
    saved = spatial.new_saved()
    spatial.forward(xd, wd, saved=saved)
    _, gw = spatial.backward(gy, saved, None, need_gx=False)
    _, gK = layer.backward(gy, saved, None, need_gx=False)
    k = torch.arange(N, dtype=torch.float64, device="cuda")
    taps = torch.arange(n, dtype=torch.float64, device="cuda")
    wave = lambda q: torch.polar(torch.ones_like(q), 2 * np.pi * q / N)  # conj(W^q)  # noqa: E731
    rows, cols = wave(taps[:, None] * k), wave(k[: N // 2 + 1, None] * taps)
    ref = torch.stack([(rows @ gK[o].to(torch.complex128) @ cols).real for o in range(S)])
    err = float((gw.double() - ref).norm() / ref.norm())
    print(f"dL/dw rounding {N}->{M} n={n}: {err:.3e}", flush=True)
    assert err < 1.18e-7

"""GPU parity of the fused CIC + FDP layer (forward and backward) and of the
multi-layer stacks, against the float64 oracle on the same seeded inputs.

The stack tests run the four synthetic CIC workloads at their full sizes, in
the same launch configuration the benchmark times (paper_2106_12736_amd.layers.CicStack),
and compare every output and every gradient element."""

import ctypes
import zlib

import numpy as np
import pytest
import torch

from _parity import assert_parity, to_np
from oracle import fdc
from paper_2106_12736_amd import _lib, inputs, layers

pytestmark = pytest.mark.gpu


def _rng(*key):
    return np.random.default_rng(zlib.crc32(repr(key).encode()))


def _gpu(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


ORACLE_MODE = {"none": fdc.ARTIFACT_NONE, "crop": fdc.ARTIFACT_CROP, "roll": fdc.ARTIFACT_ROLL}

LAYER_CASES = [
    # N, M, B, C, J, artifact, kernel_n
    (4, 2, 1, 1, 1, "none", 1),
    (4, 4, 2, 1, 3, "none", 1),
    (8, 4, 2, 2, 2, "none", 1),
    (8, 2, 1, 1, 2, "none", 1),
    (16, 8, 2, 1, 4, "crop", 3),
    (16, 16, 1, 2, 1, "roll", 3),
    (32, 16, 2, 2, 3, "none", 1),
    (32, 8, 1, 3, 2, "roll", 4),
    (64, 32, 2, 1, 4, "none", 1),
    (64, 64, 2, 2, 2, "crop", 5),
    (128, 64, 2, 2, 2, "none", 1),
    (128, 32, 1, 1, 8, "none", 1),
    (256, 128, 2, 2, 2, "none", 1),
    (256, 256, 1, 1, 3, "roll", 3),
    (512, 256, 2, 1, 8, "none", 1),
    (512, 128, 1, 2, 2, "crop", 3),
    (1024, 512, 2, 1, 8, "none", 1),
    (1024, 1024, 1, 1, 2, "none", 1),
    (1024, 256, 1, 2, 1, "none", 1),
    (224, 224, 2, 2, 2, "crop", 3),
]


@pytest.mark.parametrize("N,M,B,C,J,artifact,kn", LAYER_CASES)
def test_layer_forward_backward(N, M, B, C, J, artifact, kn):
    print(f"layer N={N} M={M} B={B} C={C} J={J} {artifact}/{kn}", flush=True)
    rng = _rng("layer", N, M, B, C, J, artifact, kn)
    S = C * J
    x = rng.random((B, C, N, N), dtype=np.float32)
    K = inputs.spectral_kernels(rng, S, N)
    layer = layers.CicLayer(B, C, S, N, M, artifact, kn)
    gy = rng.standard_normal((B, S, layer.out, layer.out), dtype=np.float32)
    saved = layer.new_saved()
    xg, Kg = _gpu(x), _gpu(K)
    y = layer.forward(xg, Kg, saved=saved)
    gx, gK = layer.backward(_gpu(gy), saved, Kg)

    mode = ORACLE_MODE[artifact]
    ry, xs = fdc.cic_fdp_layer_forward(x.astype(np.float64), K.astype(np.complex128), M, mode, kn)
    rgx, rgK = fdc.cic_fdp_layer_backward(gy.astype(np.float64), xs, K.astype(np.complex128), M, mode, kn)
    assert_parity(to_np(y), ry, "y")
    assert_parity(to_np(layer.saved_spectrum(saved)), fdc.fdp(xs, M, M), "saved spectrum")
    assert_parity(to_np(gx), rgx, "gx")
    assert_parity(to_np(gK), rgK, "gK")
    # bins dropped by FDP get exact zeros
    kept = np.zeros((N, N // 2 + 1), bool)
    kept[list(range(M // 2)) + list(range(N - M // 2, N)), : M // 2 + 1] = True
    assert np.all(to_np(gK)[:, ~kept] == 0)


# One-launch layers: every size pair; one image (no partial sums) and several; 1, 2, 4, 8 and
# 5 output channels a channel (the channels-side-by-side forms and the one-by-one form); crop
# and roll; enough planes to leave the small-launch forms.
SMALL_CASES = [
    # N, M, B, C, J, artifact, kernel_n
    (32, 32, 1, 3, 5, "crop", 7),
    (32, 32, 3, 2, 4, "roll", 5),
    (32, 16, 1, 1, 8, "none", 1),
    (32, 16, 5, 130, 1, "crop", 3),
    (32, 8, 2, 3, 2, "roll", 8),
    (32, 8, 3, 1, 4, "crop", 2),
    (64, 64, 3, 1, 4, "roll", 3),
    (64, 64, 1, 2, 1, "crop", 64),
    (64, 32, 3, 3, 8, "crop", 3),
    (64, 32, 2, 270, 2, "none", 1),
    (64, 16, 2, 2, 5, "none", 1),
    (128, 64, 2, 1, 2, "crop", 5),
    (128, 64, 3, 2, 1, "roll", 6),
    (128, 32, 1, 2, 4, "crop", 3),
    (128, 32, 3, 1, 3, "none", 1),
]


@pytest.mark.parametrize("N,M,B,C,J,artifact,kn", SMALL_CASES)
def test_small_layer(N, M, B, C, J, artifact, kn):
    """The one-launch forward and backward, each output also on its own.  Four transforms of
    log2(N) <= 7 roundings each and sums of at most 8 terms, in units of u = 6e-8 and adding
    as a random walk, stay below 12 u = 7e-7; the bound is four times that."""
    print(f"small layer N={N} M={M} B={B} C={C} J={J} {artifact}/{kn}", flush=True)
    rng = _rng("small", N, M, B, C, J, artifact, kn)
    S = C * J
    x = rng.random((B, C, N, N), dtype=np.float32)
    K = inputs.spectral_kernels(rng, S, N)
    layer = layers.CicLayer(B, C, S, N, M, artifact, kn)
    gy = rng.standard_normal((B, S, layer.out, layer.out), dtype=np.float32)
    xg, Kg, gyg = _gpu(x), _gpu(K), _gpu(gy)
    saved = layer.new_saved()
    y = layer.forward(xg, Kg, saved=saved)
    gx, gK = layer.backward(gyg, saved, Kg)
    assert torch.equal(y, layer.forward(xg, Kg))
    only_x, _ = layer.backward(gyg, None, Kg, need_gk=False)
    _, only_k = layer.backward(gyg, saved, None, need_gx=False)
    assert torch.equal(gx, only_x) and torch.equal(gK, only_k)

    mode = ORACLE_MODE[artifact]
    ry, xs = fdc.cic_fdp_layer_forward(x.astype(np.float64), K.astype(np.complex128), M, mode, kn)
    rgx, rgK = fdc.cic_fdp_layer_backward(gy.astype(np.float64), xs, K.astype(np.complex128), M, mode, kn)
    for got, ref, name in ((y, ry, "y"), (gx, rgx, "gx"), (gK, rgK, "gK")):
        assert_parity(to_np(got), ref, name, rel=3e-6)
    assert_parity(to_np(layer.saved_spectrum(saved)), fdc.fdp(xs, M, M), "saved spectrum", rel=3e-6)
    kept = np.zeros((N, N // 2 + 1), bool)
    kept[list(range(M // 2)) + list(range(N - M // 2, N)), : M // 2 + 1] = True
    assert np.all(to_np(gK)[:, ~kept] == 0)


@pytest.mark.parametrize("N,M,B,C,J", [(512, 256, 1, 1, 8), (512, 128, 2, 1, 12), (1024, 512, 1, 1, 8),
                                       (256, 128, 1, 2, 16), (512, 256, 5, 3, 8), (1024, 512, 9, 1, 8)])
def test_forward_few_planes(N, M, B, C, J):
    """The CIC inverse with an output channel per workgroup (few planes) and with four (the last
    two cases).  Four transforms of log2(N) <= 10 roundings and a product, units of 6e-8 adding
    as a random walk: below 12 u = 7e-7; the bound is four times that."""
    print(f"few planes N={N} M={M} B={B} C={C} J={J}", flush=True)
    rng = _rng("few", N, M, B, C, J)
    x = rng.random((B, C, N, N), dtype=np.float32)
    K = inputs.spectral_kernels(rng, C * J, N)
    layer = layers.CicLayer(B, C, C * J, N, M, "none", 1)
    y = layer.forward(_gpu(x), _gpu(K))
    ry, _ = fdc.cic_fdp_layer_forward(x.astype(np.float64), K.astype(np.complex128), M, ORACLE_MODE["none"], 1)
    assert_parity(to_np(y), ry, "y", rel=3e-6)


def test_layer_is_deterministic_and_reentrant():
    N, M, B, C, J = 256, 128, 4, 2, 2
    rng = _rng("det")
    x = _gpu(rng.random((B, C, N, N), dtype=np.float32))
    K = _gpu(inputs.spectral_kernels(rng, C * J, N))
    gy = _gpu(rng.standard_normal((B, C * J, M, M), dtype=np.float32))
    layer = layers.CicLayer(B, C, C * J, N, M)
    outs = []
    for _ in range(2):
        saved = layer.new_saved()
        y = layer.forward(x, K, saved=saved)
        gx, gK = layer.backward(gy, saved, K)
        outs.append((y.clone(), gx.clone(), gK.clone()))
    for a, b in zip(*outs):
        assert torch.equal(a, b)


def test_gradient_outputs_are_optional():
    N, M, B, C, J = 64, 32, 2, 2, 2
    rng = _rng("opt")
    x = _gpu(rng.random((B, C, N, N), dtype=np.float32))
    K = _gpu(inputs.spectral_kernels(rng, C * J, N))
    gy = _gpu(rng.standard_normal((B, C * J, M, M), dtype=np.float32))
    layer = layers.CicLayer(B, C, C * J, N, M)
    saved = layer.new_saved()
    layer.forward(x, K, saved=saved)
    gx_full, gK_full = layer.backward(gy, saved, K)
    gx_only, none_k = layer.backward(gy, saved, K, need_gk=False)
    none_x, gK_only = layer.backward(gy, saved, K, need_gx=False)
    assert none_k is None and none_x is None
    assert torch.equal(gx_only, gx_full) and torch.equal(gK_only, gK_full)
    y_nosave = layer.forward(x, K)  # inference: nothing saved
    assert torch.equal(y_nosave, layer.forward(x, K, saved=saved))


def test_batch_not_divisible():
    # any batch size works (the paper's implementation needed batch-divisible datasets)
    for B in (1, 3, 5):
        N, M, C, J = 32, 16, 1, 2
        rng = _rng("batch", B)
        x = rng.random((B, C, N, N), dtype=np.float32)
        K = inputs.spectral_kernels(rng, C * J, N)
        layer = layers.CicLayer(B, C, C * J, N, M)
        y = layer.forward(_gpu(x), _gpu(K))
        ry, _ = fdc.cic_fdp_layer_forward(x.astype(np.float64), K.astype(np.complex128), M)
        assert_parity(to_np(y), ry, f"y B={B}")


@pytest.mark.parametrize("wl", inputs.CIC_WORKLOADS, ids=[w.name for w in inputs.CIC_WORKLOADS])
def test_stack_full_size(wl):
    print(f"stack {wl.name}", flush=True)
    d = inputs.make_cic_stack(wl)
    stack = layers.CicStack(wl.batch, wl.sizes, wl.channels)
    Ks = [_gpu(k) for k in d.kernels]
    gin = torch.empty((wl.batch, wl.channels[0], wl.sizes[0], wl.sizes[0]), dtype=torch.float32, device="cuda")
    y = stack.forward(_gpu(d.x), Ks)
    gks = [g.clone() for g in stack.backward(_gpu(d.grad), Ks, input_grad=gin)]
    torch.cuda.synchronize()

    Kd = [k.astype(np.complex128) for k in d.kernels]
    ry, saved = fdc.cic_stack_forward(d.x.astype(np.float64), Kd, wl.sizes)
    rgks, rgx = fdc.cic_stack_backward(d.grad.astype(np.float64), saved, Kd, wl.sizes, want_input_grad=True)
    assert_parity(to_np(y), ry, "y")
    for i in range(wl.layers):
        assert_parity(to_np(gks[i]), rgks[i], f"gK layer {i}")
    assert_parity(to_np(gin), rgx, "gx input")
    # the training step skips the input-image gradient; the kernel gradients do not change
    gks2 = [g.clone() for g in stack.backward(_gpu(d.grad), Ks)]
    for a, b in zip(gks2, gks):
        assert torch.equal(a, b)


def _launch_names(f):
    buf = ctypes.create_string_buffer(1 << 14)
    _lib.call("fdc_kernel_timing_enable", 16, None)
    try:
        f()
        torch.cuda.synchronize()
        _lib.call("fdc_kernel_timing_launches", buf, len(buf))
    finally:
        _lib.call("fdc_kernel_timing_disable")
    return [line.split()[0] for line in buf.value.decode().splitlines()]


@pytest.mark.parametrize("N,M,B,C,J", [(64, 32, 4, 64, 4), (64, 64, 1, 4, 4), (64, 16, 16, 65, 5), (128, 64, 16, 20, 2),
                                       (128, 32, 1, 20, 2)])
def test_one_launch_query_names_the_launches(N, M, B, C, J):
    """fdc_cic_layer_one_launch against the launches that the two calls make."""
    layer = layers.CicLayer(B, C, C * J, N, M, "none", 1)
    x, gy = torch.zeros(B, C, N, N, device="cuda"), torch.zeros(B, C * J, M, M, device="cuda")
    K = torch.zeros(C * J, N, N // 2 + 1, dtype=torch.complex64, device="cuda")
    saved = layer.new_saved()
    fwd = _launch_names(lambda: layer.forward(x, K, saved=saved))
    bwd = _launch_names(lambda: layer.backward(gy, saved, K))
    forward, backward = layer.one_launch()
    assert (fwd == [f"small_fwd_{N}_{M}"]) == (forward == 1), fwd
    assert (bwd == [f"small_bwd_{N}_{M}"]) == (backward == 1), bwd
    assert (bwd == [f"small_bwd_{N}_{M}", "gk_reduce"]) == (backward == 2), bwd


# Forms that the number of planes decides: several images a workgroup with an uneven last range
# (1 and 4 channels at a time; M < N, where the row scratch of one stage lies on the planes of
# another), two of more channels at a time, a single range through partial sums and straight to
# gK, and all of an odd number of channels a forward workgroup.
SMALL_PLANE_CASES = [
    # N, M, B, C, J, most image ranges
    (64, 32, 9, 300, 1, 8),
    (32, 8, 5, 900, 4, 4),
    (128, 32, 7, 60, 4, 4),
    (128, 64, 7, 60, 1, 4),
    (64, 32, 2, 300, 4, 2),
    (32, 16, 3, 2, 6, 3),
    (128, 32, 2, 3, 6, 2),
    (32, 8, 1, 3, 8, 1),
    (128, 32, 1, 20, 2, 1),
    (128, 64, 2, 100, 3, 2),
    (64, 16, 8, 130, 12, 8),
]


@pytest.mark.parametrize("N,M,B,C,J,most", SMALL_PLANE_CASES)
def test_small_layer_by_planes(N, M, B, C, J, most):
    """As test_small_layer; at most 9 images more in dK's sums, 3 u of a random walk."""
    print(f"small layer planes N={N} M={M} B={B} C={C} J={J}", flush=True)
    rng = _rng("small planes", N, M, B, C, J)
    x = rng.random((B, C, N, N), dtype=np.float32)
    K = inputs.spectral_kernels(rng, C * J, N)
    layer = layers.CicLayer(B, C, C * J, N, M, "none", 1)
    assert layer.dk_ranges() <= most
    gy = rng.standard_normal((B, C * J, M, M), dtype=np.float32)
    xg, Kg, gyg = _gpu(x), _gpu(K), _gpu(gy)
    saved = layer.new_saved()
    y = layer.forward(xg, Kg, saved=saved)
    gx, gK = layer.backward(gyg, saved, Kg)
    only_x, _ = layer.backward(gyg, None, Kg, need_gk=False)
    _, only_k = layer.backward(gyg, saved, None, need_gx=False)
    assert torch.equal(gx, only_x) and torch.equal(gK, only_k)
    ry, xs = fdc.cic_fdp_layer_forward(x.astype(np.float64), K.astype(np.complex128), M, ORACLE_MODE["none"], 1)
    rgx, rgK = fdc.cic_fdp_layer_backward(gy.astype(np.float64), xs, K.astype(np.complex128), M, ORACLE_MODE["none"], 1)
    for got, ref, name in ((y, ry, "y"), (gx, rgx, "gx"), (gK, rgK, "gK")):
        assert_parity(to_np(got), ref, name, rel=3e-6)
    kept = np.zeros((N, N // 2 + 1), bool)
    kept[list(range(M // 2)) + list(range(N - M // 2, N)), : M // 2 + 1] = True
    assert np.all(to_np(gK)[:, ~kept] == 0)

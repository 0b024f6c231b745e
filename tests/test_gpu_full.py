"""GPU parity of the Full FDC layer (Algorithm 2 with the per-bin channel sum of
Eq. 2; kernel spectra generated from n x n weights as in section 2.4.1.2) and its
backward, against the float64 oracle on the same seeded inputs.

Small cases are compared element by element; they span several batch tiles, output
blocks, contraction steps and dL/dw channel blocks, each with a ragged edge.  The
six 16-image VGG-block layers (224 and 512 pixels, 64/128/256 channels) run at full
size in the same launch configuration the benchmark times, and are checked on
sampled (image, channel) slices, each of which the oracle computes on its own."""

import zlib

import numpy as np
import pytest
import torch

from _parity import assert_parity, rel_l2, to_np
from oracle import dft, fdc
from paper_2106_12736_amd import inputs, layers

pytestmark = pytest.mark.gpu

ORACLE_MODE = {"none": fdc.ARTIFACT_NONE, "crop": fdc.ARTIFACT_CROP, "roll": fdc.ARTIFACT_ROLL}


def _rng(*key):
    return np.random.default_rng(zlib.crc32(repr(key).encode()))


def _gpu(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _out_size(P, n, artifact):
    return P - n + 1 if artifact == "crop" else P


SMALL_CASES = [
    # B, Cin, Cout, P, n, artifact
    (1, 1, 1, 8, 3, "crop"),
    (2, 3, 5, 8, 3, "crop"),
    (3, 2, 4, 8, 2, "roll"),
    (17, 6, 9, 16, 3, "crop"),     # two batch tiles, ragged
    (2, 5, 300, 16, 1, "none"),    # two forward output blocks
    (2, 300, 3, 16, 3, "none"),    # two dL/dX output blocks, 75 contraction steps
    (5, 33, 40, 32, 5, "roll"),    # two dL/dw channel blocks each way
    (40, 3, 4, 16, 3, "crop"),     # three dL/dw batch chunks, ragged
    (2, 4, 4, 64, 4, "crop"),
    (16, 8, 8, 128, 3, "crop"),
    (4, 3, 5, 224, 3, "crop"),
    (2, 2, 3, 256, 3, "roll"),
    (1, 2, 2, 512, 5, "none"),
    (1, 1, 2, 1024, 3, "crop"),
]


@pytest.mark.parametrize("B,Cin,Cout,P,n,artifact", SMALL_CASES)
def test_full_layer_forward_backward(B, Cin, Cout, P, n, artifact):
    print(f"full B={B} Cin={Cin} Cout={Cout} P={P} n={n} {artifact}", flush=True)
    rng = _rng("full", B, Cin, Cout, P, n, artifact)
    O = _out_size(P, n, artifact)
    x = inputs.normal(rng, (B, Cin, P, P))
    w = inputs.he_normal_weights(rng, Cout, Cin, n)
    gy = inputs.normal(rng, (B, Cout, O, O))

    layer = layers.FullLayer(B, Cin, Cout, P, kernel_n=n, artifact=artifact)
    assert layer.out == O
    xd, wd = _gpu(x), _gpu(w)
    saved = layer.new_saved()
    y = layer.forward(xd, wd, saved=saved)
    gx, gw = layer.backward(_gpu(gy), saved, wd)
    torch.cuda.synchronize()

    mode = ORACLE_MODE[artifact]
    y_ref, xs_ref = fdc.full_fdc_forward(x.astype(np.float64), w.astype(np.float64), mode)
    gx_ref, gw_ref = fdc.full_fdc_backward(gy.astype(np.float64), xs_ref, w.astype(np.float64), mode)
    assert_parity(to_np(layer.saved_spectrum(saved)), xs_ref, "saved rfft2(x)")
    assert_parity(to_np(y), y_ref, "y")
    assert_parity(to_np(gx), gx_ref, "gx")
    assert_parity(to_np(gw), gw_ref, "gw")


# Edges of the contraction's tiles: image groups of 8 and 16 (and the rest after whole
# groups), output groups of one to four 16-output tiles and two of them, channel steps of 4,
# column groups wider than the spectrum (P = 8) or with a ragged last one (P = 224), each
# kernel size.
CONTRACT_CASES = [
    # B, Cin, Cout, P, n
    (1, 4, 16, 8, 3),
    (8, 16, 17, 16, 3),
    (9, 17, 33, 16, 3),
    (16, 33, 49, 32, 3),
    (20, 49, 65, 8, 5),
    (24, 3, 80, 16, 5),
    (25, 80, 5, 16, 1),
    (4, 33, 20, 224, 3),
    (7, 65, 18, 32, 2),
    (12, 20, 35, 64, 4),
    (6, 130, 20, 64, 5),
    (1, 35, 70, 32, 3),    # 4-image tiles: 64-output groups, the second ragged; channels past 4
    (19, 41, 64, 16, 5),   # ... after 16-image tiles
]


@pytest.mark.parametrize("B,Cin,Cout,P,n", CONTRACT_CASES)
def test_full_contraction_tiles(B, Cin, Cout, P, n):
    """Forward and dL/dX at the tile edges.  Four transforms of log2(P) <= 8 roundings each
    and a sum over at most 130 channels of products, in units of u = 6e-8 and adding as a
    random walk, stay below 20 u = 1.2e-6; the bound is four times that."""
    print(f"full contraction B={B} Cin={Cin} Cout={Cout} P={P} n={n}", flush=True)
    rng = _rng("full-tiles", B, Cin, Cout, P, n)
    x = inputs.normal(rng, (B, Cin, P, P))
    w = inputs.he_normal_weights(rng, Cout, Cin, n)
    gy = inputs.normal(rng, (B, Cout, P, P))
    layer = layers.FullLayer(B, Cin, Cout, P, kernel_n=n, artifact="roll")
    saved = layer.new_saved()
    wd = _gpu(w)
    y = layer.forward(_gpu(x), wd, saved=saved)
    gx, gw = layer.backward(_gpu(gy), saved, wd)
    torch.cuda.synchronize()
    y_ref, xs_ref = fdc.full_fdc_forward(x.astype(np.float64), w.astype(np.float64), fdc.ARTIFACT_ROLL)
    gx_ref, gw_ref = fdc.full_fdc_backward(gy.astype(np.float64), xs_ref, w.astype(np.float64), fdc.ARTIFACT_ROLL)
    assert_parity(to_np(y), y_ref, "y", rel=5e-6)
    assert_parity(to_np(gx), gx_ref, "gx", rel=5e-6)
    assert_parity(to_np(gw), gw_ref, "gw", rel=5e-6)


# Sizes past the launches of few workgroups: images by 16, by 16 and the rest in one launch, by 8
# and by 4, groups of one to four 16-output tiles and two of them, every kernel size; and few
# channels of a large spectrum, which take the form of few workgroups.
CONTRACT_LARGE_CASES = [
    # B, Cin, Cout, P, n
    (9, 17, 40, 64, 3),
    (20, 40, 40, 64, 1),
    (22, 40, 40, 64, 2),
    (22, 12, 100, 64, 4),
    (5, 40, 100, 128, 1),
    (3, 20, 64, 128, 4),
    (2, 20, 64, 128, 2),
    (4, 20, 64, 128, 1),
    (24, 18, 16, 128, 5),
    (6, 12, 30, 224, 3),
    (8, 3, 64, 128, 3),
]


@pytest.mark.parametrize("B,Cin,Cout,P,n", CONTRACT_LARGE_CASES)
def test_full_contraction_large(B, Cin, Cout, P, n):
    """As test_full_contraction_tiles, with sums over at most 100 channels."""
    test_full_contraction_tiles(B, Cin, Cout, P, n)


def test_full_weight_gradient_large_grid():
    """dL/dw of 4096 x 4096 channels: 16384 tiles x 258 bin chunks = 4.2 million workgroups of 1024
    threads, more than the 2^32 threads that HIP counts in a launch; a launch cut short leaves the last
    chunks out of every sum.  A 1 x 1 kernel scales, so dL/dw[s, c] = <gy_s, x_c>, in 64 bits for 48
    pairs in either direction.  Bound as in test_full_contraction_tiles."""
    S = C = 4096
    P = 512
    if torch.cuda.mem_get_info()[0] < 64 << 30:
        pytest.skip("64 GiB of device memory are needed")
    gen = torch.Generator(device="cuda").manual_seed(7)
    x = torch.randn(1, C, P, P, device="cuda", generator=gen)
    w = torch.randn(S, C, 1, 1, device="cuda", generator=gen)
    layer = layers.FullLayer(1, C, S, P, kernel_n=1, artifact="none")
    saved = layer.new_saved()
    y = layer.forward(x, w, saved=saved)
    rows, cols = torch.arange(0, S, 87, device="cuda"), torch.arange(C - 1, -1, -87, device="cuda")
    ref = w[rows, :, 0, 0].double() @ x[0, :, 5].double()
    got = y[0, rows, 5].double()
    assert float((got - ref).abs().max() / ref.abs().max()) < 5e-6
    del y, got, ref
    gy = torch.randn(1, S, P, P, device="cuda", generator=gen)
    _, gw = layer.backward(gy, saved, None, need_gx=False)
    ref = gy[0, rows].double().flatten(1) @ x[0, cols].double().flatten(1).t()
    assert float((gw[rows][:, cols, 0, 0].double() - ref).abs().max() / ref.abs().max()) < 5e-6


def test_full_layer_optional_outputs_and_repeatability():
    """Forward without `saved`, backward with only one of the two gradients, and
    bit-identical results on a second call (fixed reduction order)."""
    B, Cin, Cout, P, n = 3, 5, 7, 32, 3
    rng = _rng("full-optional")
    x = inputs.normal(rng, (B, Cin, P, P))
    w = inputs.he_normal_weights(rng, Cout, Cin, n)
    gy = inputs.normal(rng, (B, Cout, P - n + 1, P - n + 1))
    layer = layers.FullLayer(B, Cin, Cout, P, kernel_n=n, artifact="crop")
    xd, wd, gyd = _gpu(x), _gpu(w), _gpu(gy)
    y0 = layer.forward(xd, wd)
    saved = layer.new_saved()
    y1 = layer.forward(xd, wd, saved=saved)
    assert torch.equal(y0, y1)
    gx_only, none_w = layer.backward(gyd, None, wd, need_gw=False)
    assert none_w is None
    none_x, gw_only = layer.backward(gyd, saved, None, need_gx=False)
    assert none_x is None
    gx, gw = layer.backward(gyd, saved, wd)
    gx2, gw2 = layer.backward(gyd, saved, wd)
    torch.cuda.synchronize()
    assert torch.equal(gx_only, gx) and torch.equal(gw_only, gw)
    assert torch.equal(gx, gx2) and torch.equal(gw, gw2)
    y_ref, xs_ref = fdc.full_fdc_forward(x.astype(np.float64), w.astype(np.float64), fdc.ARTIFACT_CROP)
    gx_ref, gw_ref = fdc.full_fdc_backward(gy.astype(np.float64), xs_ref, w.astype(np.float64),
                                           fdc.ARTIFACT_CROP)
    assert_parity(to_np(y0), y_ref, "y")
    assert_parity(to_np(gx), gx_ref, "gx")
    assert_parity(to_np(gw), gw_ref, "gw")


def test_full_layer_cic_special_case():
    """With Cin = Cout = 1 and a 1 x 1 kernel the layer scales the image by w."""
    x = inputs.normal(_rng("full-1x1"), (4, 1, 64, 64))
    layer = layers.FullLayer(4, 1, 1, 64, kernel_n=1, artifact="none")
    w = torch.full((1, 1, 1, 1), -1.75, device="cuda")
    y = layer.forward(_gpu(x), w)
    torch.cuda.synchronize()
    assert_parity(to_np(y), -1.75 * x.astype(np.float64), "y")


@pytest.mark.parametrize("wl", inputs.FULL_FDC_WORKLOADS, ids=lambda w: w.name)
def test_full_layer_workload_sampled(wl):
    """Full-size layer in the benchmark's configuration; the oracle checks sampled
    slices: y[b][s], gx[b][c], saved[b][c] for sampled images b and channels, and
    gw[s][c] (a sum over the whole batch) for sampled channel pairs."""
    print(f"full workload {wl.name}", flush=True)
    d = inputs.make_full_fdc(wl)
    B, Cin, Cout, P, n = wl.batch, wl.cin, wl.cout, wl.size, wl.n
    layer = layers.FullLayer(B, Cin, Cout, P, kernel_n=n, artifact="crop")
    xd, wd, gyd = _gpu(d.x), _gpu(d.w), _gpu(d.grad)
    saved = layer.new_saved()
    y = layer.forward(xd, wd, saved=saved)
    gx, gw = layer.backward(gyd, saved, wd)
    torch.cuda.synchronize()
    print("  gpu done", flush=True)

    bs = [0, B - 1]
    ss = [0, Cout // 2 + 1, Cout - 1]
    cs = [0, Cin // 3, Cin - 1]
    x64 = d.x.astype(np.float64)
    w64 = d.w.astype(np.float64)
    g64 = d.grad.astype(np.float64)
    crop = fdc.ARTIFACT_CROP
    for b in bs:
        # forward slice y[b][ss] needs every input channel of image b
        y_ref, xs_b = fdc.full_fdc_forward(x64[b:b + 1], w64[ss], crop)
        assert_parity(to_np(y[b, ss]), y_ref[0], f"y[{b}]")
        assert_parity(to_np(layer.saved_spectrum(saved)[b, cs]), xs_b[0, cs], f"saved[{b}]")
        # dL/dx slice gx[b][cs] needs every output channel of image b
        gx_ref, _ = fdc.full_fdc_backward(g64[b:b + 1], xs_b[:, cs], w64[:, cs], crop)
        assert_parity(to_np(gx[b, cs]), gx_ref[0], f"gx[{b}]")
    # dL/dw slice gw[ss2][cs2] needs every image of the batch; the pairs straddle the
    # 16- and 32-channel tile borders of the dL/dw kernel and reach both ends
    ss2 = sorted({0, 15, 16, 31, 32, Cout // 2 + 1, Cout - 33, Cout - 1})
    cs2 = sorted({0, 16, 31, 32, Cin // 3, Cin - 1})
    xs_c = dft.rfft2(x64[:, cs2])
    _, gw_ref = fdc.full_fdc_backward(g64[:, ss2], xs_c, w64[ss2][:, cs2], crop, want_gx=False)
    assert_parity(to_np(gw[ss2][:, cs2]), gw_ref, "gw")
    assert torch.isfinite(y).all() and torch.isfinite(gx).all() and torch.isfinite(gw).all()
    # every element at once: the layer is linear in w and in x, so <gw, w> = <gy, y> = <gx, x>
    # (Euler's identity for linear maps; float64 sums of the GPU's own tensors)
    yy = float((to_np(y).astype(np.float64) * g64).sum())
    ww = float((to_np(gw).astype(np.float64) * w64).sum())
    xx = float((to_np(gx).astype(np.float64) * x64).sum())
    scale = float(np.sqrt((to_np(y).astype(np.float64) ** 2).sum() * (g64 ** 2).sum()))
    assert abs(ww - yy) <= 1e-4 * scale, ("<gw, w> != <gy, y>", ww, yy, scale)
    assert abs(xx - yy) <= 1e-4 * scale, ("<gx, x> != <gy, y>", xx, yy, scale)


@pytest.mark.parametrize("B,n", [(9, 3), (8, 2), (4, 5)])
def test_full_weight_gradient_rounding(B, n):
    """dL/dw is off by little more than the rounding of the float32 transforms it is formed from,
    which is measured here: the same sums in float64 over float32 spectra.  Products and sums
    add up to 2 B roundings a bin (twice that in the three-product form) and 2 P / 8 in a wave's
    columns, 2 (2 B) / 2 + 32 / 2 <= 34 as partial sums grow like a random walk, of 2.5e-8 each
    (root mean square of 2^-24 over a binade): below 1.5e-7.  Row pairs added up in float32
    as well gave 1.6e-7 to 1.9e-7."""
    C, S, P = 24, 40, 128
    whole = alone = 0.0
    for seed in range(2):
        rng = _rng("gw rounding", B, n, seed)
        x, gy = inputs.normal(rng, (B, C, P, P)), inputs.normal(rng, (B, S, P, P))
        w = inputs.he_normal_weights(rng, S, C, n)
        layer = layers.FullLayer(B, C, S, P, kernel_n=n, artifact="roll")
        saved = layer.new_saved()
        layer.forward(_gpu(x), _gpu(w), saved=saved)
        gw = to_np(layer.backward(_gpu(gy), saved, _gpu(w))[1])
        shift = ((n - 1) // 2, (n - 1) // 2)
        rolled = np.roll(gy, shift, (-2, -1))

        def sums(X, G):
            D = np.matmul(G.reshape(B, S, -1).transpose(2, 1, 0), X.reshape(B, C, -1).transpose(2, 0, 1).conj())
            return np.fft.irfft2(D.transpose(1, 2, 0).reshape(S, C, P, P // 2 + 1))[..., :n, :n]

        ref = sums(np.fft.rfft2(x.astype(np.float64)), np.fft.rfft2(rolled.astype(np.float64)))
        X, G = (to_np(layers.FftPlan(B * k, P, P).rfft2(_gpu(t))).reshape(B, k, P, P // 2 + 1).astype(np.complex128)
                for t, k in ((x, C), (rolled, S)))
        whole += rel_l2(gw, ref) / 2
        alone += rel_l2(sums(X, G), ref) / 2
    added = np.sqrt(max(0.0, whole**2 - alone**2))
    print(f"dL/dw B={B} n={n}: {whole:.3e}, transforms {alone:.3e}, sums {added:.3e}", flush=True)
    assert added < 1.5e-7

"""GPU parity of the register-staged kernels, which run the tensors that a
buffer resource cannot address (2 GiB and more): every tile, weight layout,
slice kind and split of the data convolutions, and the kernel gradients.

The forward pass and the kernel gradient read x from a channel slice of a
buffer whose pixel stride takes the span past 2 GiB, so that the layers
themselves stay small. The other passes read dense tensors: 2 GiB of output
gradient (or, transposed, of input) with many channels, drawn on the device;
the oracle gets bands of rows at the image's top, middle and bottom, whose
inner rows depend on nothing else.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_1909_11150_amd as fg
import synth
from gpu_util import conv_parity, dev, empty16, host, sample_indices, workspace

pytestmark = pytest.mark.gpu

FWD, DX, DW, CT = fg.OP_FWD, fg.OP_BWD_DATA, fg.OP_BWD_WEIGHT, fg.OP_CONVT
SPAN = 1 << 30   # elements: 2 GiB
SMALL, BIG = "Cfg<128, 128, 2, 2>", "Cfg<256, 256, 2, 4>"


def _data(cfg, wk, whole, split):
    b = lambda v: "true" if v else "false"
    return f"data_conv_staged_kernel<{cfg}, {b(wk)}, {b(whole)}, {b(split)}>"


# (n, h, w, c, k, r, stride, pad): the forward kernel
FORWARD = [
    ((2, 67, 69, 16, 24, 3, 2, 1), _data(SMALL, True, False, False)),
    ((3, 73, 38, 48, 16, 3, 1, 1), _data(SMALL, True, False, True)),
    ((2, 82, 55, 64, 16, 1, 1, 0), _data(SMALL, True, True, False)),
    ((2, 59, 82, 64, 16, 3, 1, 1), _data(SMALL, True, True, True)),
    ((3, 76, 85, 16, 408, 1, 1, 0), _data(BIG, True, False, False)),
    ((2, 79, 55, 336, 400, 3, 1, 1), _data(BIG, True, False, True)),
    ((3, 81, 78, 128, 464, 1, 1, 0), _data(BIG, True, True, False)),
    ((2, 69, 67, 256, 392, 3, 1, 1), _data(BIG, True, True, True)),
]
# the kernel gradient
GRADIENT = [
    ((1, 15, 20, 24, 40, 3, 1, 1), f"wgrad_staged_kernel<{SMALL}, false>"),
    ((2, 67, 69, 16, 24, 3, 2, 1), f"wgrad_staged_kernel<{SMALL}, true>"),
    ((1, 15, 20, 40, 264, 3, 1, 1), f"wgrad_staged_kernel<{BIG}, false>"),
    ((2, 77, 57, 32, 256, 3, 1, 1), f"wgrad_staged_kernel<{BIG}, true>"),
]
# the input gradient, dy past 2 GiB
INPUT_GRADIENT = [
    ((1, 3995, 192, 16, 1400, 3, 1, 1), _data(SMALL, False, False, False)),
    ((1, 2456, 173, 16, 2528, 1, 1, 0), _data(SMALL, False, False, True)),
    ((1, 3708, 181, 16, 1600, 1, 1, 0), _data(SMALL, False, True, False)),
    ((1, 2797, 150, 16, 2560, 1, 1, 0), _data(SMALL, False, True, True)),
    ((1, 3561, 177, 256, 1704, 1, 1, 0), _data(BIG, False, False, False)),
    ((1, 743, 196, 256, 7376, 1, 1, 0), _data(BIG, False, False, True)),
    ((1, 3364, 172, 256, 1856, 1, 1, 0), _data(BIG, False, True, False)),
    ((1, 1692, 87, 256, 7296, 3, 1, 1), _data(BIG, False, True, True)),
]
# transposed convolutions, x past 2 GiB: (n, h, w, c_in, c_out)
TRANSPOSED = [
    ((1, 3567, 192, 1568, 16), _data(SMALL, False, False, False)),
    ((1, 1695, 165, 3840, 16), _data(SMALL, False, True, True)),
]


def _x_ld(shape):
    """The least pixel stride that takes the input's span past 2 GiB."""
    npix = shape[0] * shape[1] * shape[2]
    ld = (SPAN // (npix - 1) // 8 + 1) * 8
    assert npix * ld < 2 * SPAN
    return ld


def descs():
    """(descriptor, pass, kernel) of every case (also read by the CPU tests)."""
    for cases, op in ((FORWARD, FWD), (GRADIENT, DW), (INPUT_GRADIENT, DX)):
        for s, kern in cases:
            n, h, w, c, k, r, st, pd = s
            yield (fg.ConvDesc.make(n, h, w, c, k, r, r, st, pd,
                                    x_ld=0 if op == DX else _x_ld(s)), op, kern)
    for (n, h, w, c, k), kern in TRANSPOSED:
        yield fg.ConvDesc.make(n, h, w, c, k, 4, 4, 2, 1), CT, kern


def test_every_staged_kernel_is_named():
    want = {_data(cfg, wk, whole, split) for cfg in (SMALL, BIG) for wk in (False, True)
            for whole in (False, True) for split in (False, True)}
    want |= {f"wgrad_staged_kernel<{cfg}, {s}>" for cfg in (SMALL, BIG)
             for s in ("false", "true")}
    assert {k for _, _, k in descs()} == want


def _sliced(x, ld):
    """x in channels 8.. of a buffer with pixel stride ld; the rest NaN where
    a kernel could reach it by a small slip, else as allocated."""
    n, h, w, c = x.shape
    buf = torch.empty((n * h * w, ld), dtype=torch.float16, device="cuda")
    buf[:, :c + 64] = float("nan")
    buf[:, 8:8 + c] = dev(x).view(n * h * w, c)
    return buf, buf.view(-1)[8:]


@pytest.mark.parametrize("shape,kern", FORWARD, ids=[k for _, k in FORWARD])
def test_forward(shape, kern):
    n, h, w, c, k, r, st, pd = shape
    ld = _x_ld(shape)
    d = fg.ConvDesc.make(n, h, w, c, k, r, r, st, pd, x_ld=ld)
    assert fg.kernel_name(d, FWD) == kern
    rng = np.random.default_rng(sum(shape))
    x = synth.uniform(rng, (n, h, w, c))
    W = synth.normal(rng, (k, r, r, c), np.sqrt(2.0 / (r * r * c)))
    p, q = fg.out_dims(d)
    buf, xs = _sliced(x, ld)
    outs = []
    for _ in range(2):
        y = empty16((n, p, q, k))
        fg.conv2d_fwd(d, xs, dev(W), y, fg.EPI_RELU, None, workspace(d, FWD))
        outs.append(host(y))
    np.testing.assert_array_equal(outs[0].view(np.uint16), outs[1].view(np.uint16))
    idx = sample_indices(outs[0].shape, 2500, rng)
    ref = oracle.relu(oracle.conv2d_fwd_points(x, W, idx, st, pd))
    conv_parity(outs[0].ravel()[idx], ref, f"fwd {shape}")
    # added to what the output holds, in a slice of its own
    ldo = k + 24
    d.y_ld = ldo
    old = synth.normal(rng, (n * p * q, ldo))
    big = dev(old)
    fg.conv2d_fwd(d, xs, dev(W), big.view(-1)[8:], fg.EPI_ACC, None, workspace(d, FWD))
    got = host(big)
    keep = np.r_[0:8, 8 + k:ldo]
    np.testing.assert_array_equal(got[:, keep].view(np.uint16), old[:, keep].view(np.uint16))
    ref = oracle.conv2d_fwd_points(x, W, idx, st, pd)
    conv_parity(got[:, 8:8 + k].ravel()[idx],
                ref + old[:, 8:8 + k].ravel()[idx].astype(np.float64), f"acc {shape}")


@pytest.mark.parametrize("shape,kern", GRADIENT, ids=[k for _, k in GRADIENT])
def test_kernel_gradient(shape, kern):
    n, h, w, c, k, r, st, pd = shape
    ld = _x_ld(shape)
    d = fg.ConvDesc.make(n, h, w, c, k, r, r, st, pd, x_ld=ld)
    assert fg.kernel_name(d, DW) == kern
    rng = np.random.default_rng(sum(shape) + 1)
    p, q = fg.out_dims(d)
    x, dy = synth.uniform(rng, (n, h, w, c)), synth.uniform(rng, (n, p, q, k))
    buf, xs = _sliced(x, ld)
    dyd, ws = dev(dy), workspace(d, DW)
    dw, flag = empty16((k, r, r, c)), torch.zeros(1, dtype=torch.int32, device="cuda")
    fg.conv2d_bwd_weight(d, xs, dyd, dw, ws)
    ref = oracle.conv2d_bwd_weight(x, dy, r, r, st, pd)
    conv_parity(host(dw), ref, f"dW {shape}")
    checked = empty16(dw.shape)
    fg.conv2d_bwd_weight_checked(d, xs, dyd, checked, flag, ws)
    assert torch.equal(checked.view(torch.int16), dw.view(torch.int16))
    assert int(host(flag)[0]) == 0
    dyd[..., k // 2] = 60000.0        # x is not all zeros: some sum overflows
    fg.conv2d_bwd_weight_checked(d, xs, dyd, checked, flag, ws)
    assert int(host(flag)[0]) == int(not bool(torch.isfinite(checked).all())) == 1


def _device_normal(shape, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    return torch.randn(shape, dtype=torch.float16, device="cuda", generator=gen)


def _band_indices(rows, shape, rng):
    """Sampled flat indices of the given rows of a crop of one image."""
    _, m, w, ch = shape
    i = rng.integers(rows[0] * w * ch, rows[1] * w * ch, size=1000)
    edge = [(r * w + s) * ch + e for r in (rows[0], rows[1] - 1) for s in (0, w - 1)
            for e in (0, ch - 1)]
    return np.unique(np.concatenate([i, edge]))


def _bands(h):
    """(first row, end) of bands of rows, and of their rows that depend on no
    other: at the top, in the middle, and at the bottom."""
    m = 6
    return [((0, m), (0, m - 2)), ((h // 2, h // 2 + m), (h // 2 + 2, h // 2 + m - 2)),
            ((h - m, h), (h - m + 2, h))]


@pytest.mark.parametrize("shape,kern", INPUT_GRADIENT, ids=[k for _, k in INPUT_GRADIENT])
def test_input_gradient(shape, kern):
    n, h, w, c, k, r, st, pd = shape
    d = fg.ConvDesc.make(n, h, w, c, k, r, r, st, pd)
    assert fg.kernel_name(d, DX) == kern and n * h * w * k >= SPAN
    rng = np.random.default_rng(sum(shape))
    W = synth.normal(rng, (k, r, r, c), np.sqrt(1.0 / (r * r * k)))
    dy = _device_normal((n, h, w, k), 5)
    gate = _device_normal((n, h, w, c), 6)
    dx = empty16((n, h, w, c))
    fg.conv2d_bwd_data(d, dy, dev(W), dx, fg.EPI_GATE, gate, workspace(d, DX))
    for (a, b), (i, j) in _bands(h):
        idx = _band_indices((i - a, j - a), (n, b - a, w, c), rng)
        ref = oracle.conv2d_bwd_data_points(host(dy[:, a:b]), W, (n, b - a, w, c), idx, st, pd)
        ref = oracle.relu_grad(ref, host(gate[:, a:b]).ravel()[idx])
        conv_parity(host(dx[:, a:b]).ravel()[idx], ref, f"dx {shape} rows {i}..{j}")


@pytest.mark.parametrize("shape,kern", TRANSPOSED, ids=[k for _, k in TRANSPOSED])
def test_transposed(shape, kern):
    n, h, w, c, k = shape
    d = fg.ConvDesc.make(n, h, w, c, k, 4, 4, 2, 1)
    assert fg.kernel_name(d, CT) == kern and n * h * w * c >= SPAN
    rng = np.random.default_rng(sum(shape))
    Wt = synth.normal(rng, (c, 4, 4, k), np.sqrt(2.0 / (4 * c)))
    x = _device_normal((n, h, w, c), 7)
    y = empty16((n, 2 * h, 2 * w, k))
    fg.conv_transpose2d_fwd(d, x, dev(Wt), y, fg.EPI_RELU, None, workspace(d, CT))
    for (a, b), (i, j) in _bands(h):
        idx = _band_indices((2 * (i - a), 2 * (j - a)), (n, 2 * (b - a), 2 * w, k), rng)
        ref = oracle.relu(oracle.conv_transpose2d_fwd_points(host(x[:, a:b]), Wt, idx, 2, 1))
        conv_parity(host(y[:, 2 * a:2 * b]).ravel()[idx], ref, f"convT {shape} rows {i}..{j}")

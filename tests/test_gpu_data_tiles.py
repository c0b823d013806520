"""Data convolutions at the edges of the small tiles: outputs smaller than a
tile and just past one, channel counts that stages straddle taps with, parts of
a sum folded in one workgroup (also ending within a stage), output phases that
no tap reaches, operands at element offsets that are not 16-byte aligned, and
slices written or added to. Checked against the oracle, twice for the same bits."""
import numpy as np
import pytest
import torch

import oracle
import paper_1909_11150_amd as fg
import synth
from gpu_util import conv_parity, dev, host, sample_indices, workspace

pytestmark = pytest.mark.gpu

FWD, DX, CT = fg.OP_FWD, fg.OP_BWD_DATA, fg.OP_CONVT

# op, (n, h, w, c, k, r, stride, pad)
CASES = [
    (FWD, (1, 1, 1, 8, 8, 1, 1, 0)),        # one output position
    (FWD, (1, 8, 8, 16, 16, 3, 1, 1)),      # 64 positions: one tile
    (FWD, (1, 5, 13, 24, 72, 3, 1, 1)),     # 65 positions, 72 channels
    (FWD, (1, 200, 150, 48, 24, 3, 1, 1)),  # 30000 positions, stages across taps
    (FWD, (2, 40, 33, 96, 160, 4, 2, 1)),   # 96 channels: 64-deep stages across taps
    (FWD, (2, 100, 100, 128, 256, 3, 1, 1)),  # parts folded
    (FWD, (1, 64, 64, 512, 512, 3, 1, 1)),    # parts folded, 2 of 72 stages
    (FWD, (1, 24, 24, 768, 384, 3, 1, 1)),    # split, parts that end within a stage
    (FWD, (5, 17, 42, 584, 152, 3, 1, 1)),    # split, stages across taps
    (FWD, (8, 32, 32, 136, 520, 1, 1, 0)),
    (DX, (1, 1, 1, 8, 8, 1, 1, 0)),
    (DX, (3, 11, 13, 24, 40, 3, 1, 1)),
    (DX, (2, 31, 33, 64, 96, 3, 2, 1)),     # phases of different sizes and taps
    (DX, (1, 9, 10, 16, 8, 1, 2, 0)),       # phases that no tap reaches
    (DX, (2, 88, 88, 192, 160, 3, 1, 1)),
    (DX, (3, 64, 60, 264, 200, 3, 1, 1)),
    (CT, (1, 1, 1, 8, 8, 4, 2, 1)),
    (CT, (3, 7, 9, 40, 24, 4, 2, 1)),
    (CT, (2, 40, 14, 536, 320, 4, 2, 1)),   # parts folded, stages across taps
    (CT, (8, 32, 32, 256, 128, 4, 2, 1)),
]


def _tensors(op, shape, rng):
    n, h, w, c, k, r, st, pd = shape
    d = fg.ConvDesc.make(n, h, w, c, k, r, r, st, pd)
    p, q = fg.out_dims(d, op == CT)
    W = synth.normal(rng, (c, r, r, k) if op == CT else (k, r, r, c),
                     np.sqrt(2.0 / (r * r * max(c, k))))
    a = synth.uniform(rng, (n, p, q, k) if op == DX else (n, h, w, c))
    return d, a, W, (n, h, w, c) if op == DX else (n, p, q, k)


def _run(op, d, a, w, out, epi, gate=None):
    f = {FWD: fg.conv2d_fwd, DX: fg.conv2d_bwd_data, CT: fg.conv_transpose2d_fwd}[op]
    f(d, a, w, out, epi, gate, workspace(d, op))


def _ref(op, a, W, shape, oshape, idx):
    st, pd = shape[6], shape[7]
    if op == FWD:
        return oracle.conv2d_fwd_points(a, W, idx, st, pd)
    if op == DX:
        return oracle.conv2d_bwd_data_points(a, W, oshape, idx, st, pd)
    return oracle.conv_transpose2d_fwd_points(a, W, idx, st, pd)


def _at(t, off):
    """The tensor's values at element offset off of a larger buffer."""
    buf = torch.zeros(t.numel() + 16, dtype=torch.float16, device="cuda")
    v = buf[off:off + t.numel()].view(t.shape)
    v.copy_(t)
    return v


@pytest.mark.parametrize("op,shape", CASES, ids=[f"{['fwd', 'dx', '', 'convT'][o]}-{s}"
                                                 for o, s in CASES])
def test_small_tiles(op, shape):
    rng = np.random.default_rng(sum(shape) + op)
    d, a, W, oshape = _tensors(op, shape, rng)
    gate = synth.uniform(rng, oshape)
    ad, wd, gd = dev(a), dev(W), dev(gate)
    idx = sample_indices(oshape, 2500, rng)
    ref = _ref(op, a, W, shape, oshape, idx)
    outs = []
    for off in (0, 0, 1):  # the last: every pointer 2 bytes past 16-byte alignment
        out = _at(torch.full(oshape, float("nan"), dtype=torch.float16, device="cuda"), off)
        if op == DX:
            _run(op, d, _at(ad, off), _at(wd, off), out, fg.EPI_GATE, _at(gd, off))
        else:
            _run(op, d, _at(ad, off), _at(wd, off), out, fg.EPI_RELU)
        outs.append(host(out))
    want = np.where(gate.ravel()[idx].astype(np.float64) > 0, ref, 0.0) if op == DX \
        else oracle.relu(ref)
    conv_parity(outs[0].ravel()[idx], want, f"{op} {shape}")
    for o in outs[1:]:
        np.testing.assert_array_equal(outs[0].view(np.uint16), o.view(np.uint16))


@pytest.mark.parametrize("op,shape", [CASES[2], CASES[5], CASES[11], CASES[14], CASES[18]],
                         ids=str)
def test_small_tiles_add_into_a_slice(op, shape):
    """FG_EPI_ACC into channels 8.. of a wider buffer: the old value plus the
    result, rounded once; the other channels are kept."""
    rng = np.random.default_rng(sum(shape) + 7)
    d, a, W, oshape = _tensors(op, shape, rng)
    ch, npix = oshape[3], int(np.prod(oshape[:3]))
    ld = ch + 24
    if op == DX:
        d.x_ld = ld
    else:
        d.y_ld = ld
    old = synth.normal(rng, (npix, ld))
    big = dev(old)
    _run(op, d, dev(a), dev(W), big.view(-1)[8:], fg.EPI_ACC)
    got = host(big)
    keep = np.ones(ld, bool)
    keep[8:8 + ch] = False
    np.testing.assert_array_equal(got[:, keep].view(np.uint16), old[:, keep].view(np.uint16))
    idx = sample_indices(oshape, 2500, rng)
    ref = _ref(op, a, W, shape, oshape, idx) + old[:, 8:8 + ch].ravel()[idx].astype(np.float64)
    conv_parity(got[:, 8:8 + ch].ravel()[idx], ref, "acc")

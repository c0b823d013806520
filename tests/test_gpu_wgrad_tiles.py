"""Kernel gradients at the edges of their tiles: channel counts that no tile
divides (so that a tile straddles taps and runs past the last row or column),
reductions shorter than a stage, not a multiple of one, and split, on each
tile size; checked against the oracle, twice for identical bits, and once more
on operands that are not 16-byte aligned."""
import numpy as np
import pytest
import torch

import oracle
import paper_1909_11150_amd as fg
import synth
from gpu_util import conv_parity, dev, empty16, host, sample_indices, workspace

pytestmark = pytest.mark.gpu

# (n, h, w, c, k, r, stride, pad)
CASES = [
    (1, 1, 3, 8, 8, 1, 1, 0),         # three positions
    (1, 9, 7, 8, 8, 3, 1, 1),         # 63 positions: one short stage
    (1, 5, 13, 24, 72, 3, 1, 1),      # 65 positions: one row in the second stage
    (2, 13, 11, 40, 72, 3, 1, 1),     # 64-row tiles across taps
    (3, 20, 21, 72, 136, 3, 2, 1),
    (2, 17, 19, 16, 8, 4, 2, 1),      # 16 taps, 8 columns
    (3, 37, 41, 96, 160, 3, 1, 1),    # split
    (1, 1, 400, 136, 136, 1, 1, 0),   # one image row
    (5, 40, 1, 64, 200, 3, 1, 1),     # one column: every stage wraps rows
    (8, 64, 64, 128, 128, 3, 1, 1),   # 128-row tiles, split
    (2, 15, 17, 1000, 1000, 3, 1, 1),  # 256-row tiles, ragged both ways
    (1, 64, 64, 520, 264, 3, 1, 1),
    (4, 50, 46, 776, 768, 1, 1, 0),
    (1, 24, 24, 512, 256, 3, 1, 1),   # multiples of 256 on small tiles
]


def _at(t, off):
    """The tensor's values at element offset off of a larger buffer."""
    buf = torch.zeros(t.numel() + 16, dtype=torch.float16, device="cuda")
    v = buf[off:off + t.numel()].view(t.shape)
    v.copy_(t)
    return v


@pytest.mark.parametrize("shape", CASES, ids=[str(s) for s in CASES])
def test_kernel_gradient_tiles(shape):
    n, h, w, c, k, r, st, pd = shape
    d = fg.ConvDesc.make(n, h, w, c, k, r, r, st, pd)
    p, q = fg.out_dims(d)
    rng = np.random.default_rng(h * w + 7 * c + k)
    x = synth.uniform(rng, (n, h, w, c))
    dy = synth.uniform(rng, (n, p, q, k))
    xd, dyd = dev(x), dev(dy)
    outs = []
    for off in (0, 0, 1):  # the last: every pointer 2 bytes past 16-byte alignment
        dw = _at(empty16((k, r, r, c)), off)
        fg.conv2d_bwd_weight(d, _at(xd, off), _at(dyd, off), dw, workspace(d, fg.OP_BWD_WEIGHT))
        outs.append(host(dw))
    for o in outs[1:]:
        np.testing.assert_array_equal(outs[0].view(np.uint16), o.view(np.uint16))
    idx = sample_indices((k, r, r, c), 2500, rng)
    ref = oracle.conv2d_bwd_weight_points(x, dy, r, r, idx, st, pd)
    conv_parity(outs[0].ravel()[idx], ref, f"dW {shape}")

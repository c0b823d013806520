"""Gradients on the least workspace they accept: the plan in fewer parts, within
it, against the oracle; twice for the same bits, nothing written past the size,
and the plan of a full workspace unchanged by the calls between."""
import numpy as np
import pytest
import torch

import oracle
import paper_1909_11150_amd as fg
import synth
from gpu_util import conv_parity, dev, empty16, host, sample_indices, workspace
from test_abi_cpu import LEAST_OF_TWO_WS, LEAST_WS

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,op,least,full", LEAST_WS, ids=str)
def test_least_workspace(shape, op, least, full):
    n, h, w, c, k, r, st, pd = shape
    d = fg.ConvDesc.make(n, h, w, c, k, r, r, st, pd)
    p, q = fg.out_dims(d)
    rng = np.random.default_rng(sum(shape))
    x, dy = synth.uniform(rng, (n, h, w, c)), synth.uniform(rng, (n, p, q, k))
    W = synth.normal(rng, (k, r, r, c), np.sqrt(2.0 / (r * r * c)))
    oshape = W.shape if op == fg.OP_BWD_WEIGHT else x.shape
    idx = sample_indices(oshape, 2500, rng)
    if op == fg.OP_BWD_WEIGHT:
        ref = oracle.conv2d_bwd_weight_points(x, dy, r, r, idx, st, pd)
    else:
        ref = oracle.conv2d_bwd_data_points(dy, W, x.shape, idx, st, pd)
    xd, dyd, wd = dev(x), dev(dy), dev(W)
    guard = 4096
    buf = torch.empty(full + guard, dtype=torch.uint8, device="cuda")

    def run(nbytes):
        buf.fill_(0x5A)
        out = empty16(oshape)
        ws = buf[:nbytes] if nbytes else None
        if op == fg.OP_BWD_WEIGHT:
            fg.conv2d_bwd_weight(d, xd, dyd, out, ws)
        else:
            fg.conv2d_bwd_data(d, dyd, wd, out, fg.EPI_NONE, None, ws)
        assert bool((buf[nbytes:] == 0x5A).all())
        return host(out).view(np.uint16)

    first, small, whole = run(full), run(least), run(full)
    np.testing.assert_array_equal(first, whole)
    np.testing.assert_array_equal(small, run(full - 1))   # one plan below the full size
    for got in (whole, small):
        conv_parity(got.view(np.float16).ravel()[idx], ref, f"{shape} {op}")


@pytest.mark.parametrize("shape,least,mid,full", LEAST_OF_TWO_WS, ids=str)
def test_both_smaller_workspaces(shape, least, mid, full):
    """Three plans, by what the call brings: each against the oracle, nothing
    written past the size, and one plan between two of the sizes."""
    n, h, w, c, k, r, st, pd = shape
    d = fg.ConvDesc.make(n, h, w, c, k, r, r, st, pd)
    p, q = fg.out_dims(d)
    rng = np.random.default_rng(sum(shape))
    x, dy = synth.uniform(rng, (n, h, w, c)), synth.uniform(rng, (n, p, q, k))
    oshape = (k, r, r, c)
    idx = sample_indices(oshape, 2500, rng)
    ref = oracle.conv2d_bwd_weight_points(x, dy, r, r, idx, st, pd)
    xd, dyd = dev(x), dev(dy)
    buf = torch.empty(full + 4096, dtype=torch.uint8, device="cuda")

    def run(nbytes):
        buf.fill_(0x5A)
        out = empty16(oshape)
        fg.conv2d_bwd_weight(d, xd, dyd, out, buf[:nbytes])
        assert bool((buf[nbytes:] == 0x5A).all())
        return host(out).view(np.uint16)

    for lo, hi in ((least, mid - 1), (mid, full - 1), (full, full + 4096)):
        got = run(lo)
        np.testing.assert_array_equal(got, run(hi))
        conv_parity(got.view(np.float16).ravel()[idx], ref, f"{shape} {lo}")

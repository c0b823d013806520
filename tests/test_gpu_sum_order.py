"""The order of a forward or transposed pass's sums is a property of the shape:
a pass that folds the parts of its sum in one workgroup gives the bits of one
that splits them across workgroups and adds the partials in a second launch.

The plan depends on the number of images, an image's result does not: each
case runs the same images in two batches, one planned folded, the other split
into as many parts (read off its workspace), and compares every bit. Inputs are
random, so a part that ended one 16-deep step early or late would show; the
last test sees that a different number of parts does.
"""
import numpy as np
import pytest

import paper_1909_11150_amd as fg
import synth
from gpu_util import dev, empty16, host, workspace

pytestmark = pytest.mark.gpu

FWD, CT = fg.OP_FWD, fg.OP_CONVT

# pass, (h, w, c, k, r, stride, pad), images folded, images split, parts, kernels
CASES = [
    (FWD, (17, 50, 128, 24, 3, 1, 1), 6, 1, 5, "fold_kernel<64, true, false>",
     "dma_kernel<64, true, true>"),
    (FWD, (29, 18, 320, 368, 3, 1, 1), 4, 3, 5, "fold_kernel<64, true, false>",
     "dma_kernel<128, true, true>"),
    (FWD, (17, 7, 776, 32, 1, 1, 0), 6, 1, 4, "fold_kernel<64, true, true>",
     "gen_kernel<64, true, true>"),
    (FWD, (14, 55, 352, 400, 3, 1, 1), 6, 8, 5, "fold_kernel<64, true, true>",
     "dma_kernel<true, true>"),
    (FWD, (51, 19, 320, 264, 3, 1, 1), 6, 2, 5, "fold_kernel<64x128, true, false>",
     "dma_kernel<128, true, true>"),
    (FWD, (27, 41, 104, 72, 3, 1, 1), 8, 1, 4, "fold_kernel<64x128, true, true>",
     "gen_kernel<64, true, true>"),
    (FWD, (19, 54, 112, 80, 3, 1, 1), 8, 2, 4, "fold_kernel<64x128, true, true>",
     "gen_kernel<64x128, true, true>"),
    (FWD, (26, 30, 320, 352, 3, 1, 1), 8, 2, 5, "fold_kernel<128, true, false>",
     "dma_kernel<128, true, true>"),
    (FWD, (39, 59, 224, 240, 3, 1, 1), 8, 2, 3, "fold_kernel<128, true, true>",
     "gen_kernel<128, true, true>"),
    (CT, (31, 6, 256, 16, 4, 2, 1), 8, 1, 4, "fold_kernel<64, false, false>",
     "dma_kernel<64, false, true>"),
    (CT, (5, 5, 184, 24, 4, 2, 1), 3, 1, 3, "fold_kernel<64, false, true>",
     "gen_kernel<64, false, true>"),
    (CT, (10, 18, 792, 448, 4, 2, 1), 3, 8, 5, "fold_kernel<64, false, true>",
     "gen_kernel<false, true>"),
    (CT, (34, 59, 704, 32, 4, 2, 1), 6, 1, 4, "fold_kernel<64x128, false, false>",
     "dma_kernel<64x128, false, true>"),
    (CT, (58, 16, 296, 16, 4, 2, 1), 6, 1, 5, "fold_kernel<64x128, false, true>",
     "gen_kernel<64x128, false, true>"),
    (CT, (51, 41, 512, 80, 4, 2, 1), 4, 1, 3, "fold_kernel<128, false, false>",
     "dma_kernel<128, false, true>"),
    (CT, (17, 69, 416, 72, 4, 2, 1), 7, 2, 3, "fold_kernel<128/32, false, false>",
     "dma_kernel<128/32, false, true>"),
    (CT, (18, 53, 456, 144, 4, 2, 1), 4, 3, 2, "fold_kernel<128, false, true>",
     "gen_kernel<128, false, true>"),
]


def desc(op, n, shape):
    h, w, c, k, r, st, pd = shape
    return fg.ConvDesc.make(n, h, w, c, k, r, r, st, pd)


def parts_of_split(op, n, shape):
    """Parts that a split pass's workspace holds (0: not split)."""
    d = desc(op, n, shape)
    p, q = fg.out_dims(d, op == CT)
    return fg.workspace_bytes(d, op) // (4 * n * p * q * d.k)


def _inputs(op, n, shape):
    h, w, c, k, r, _, _ = shape
    rng = np.random.default_rng(sum(shape))
    wshape = (c, r, r, k) if op == CT else (k, r, r, c)
    return (synth.uniform(rng, (n, h, w, c)),
            synth.normal(rng, wshape, np.sqrt(2.0 / (r * r * c))))


def _run(op, n, shape, x, W):
    d = desc(op, n, shape)
    p, q = fg.out_dims(d, op == CT)
    y = empty16((n, p, q, d.k))
    f = fg.conv_transpose2d_fwd if op == CT else fg.conv2d_fwd
    f(d, dev(x[:n]), dev(W), y, fg.EPI_NONE, None, workspace(d, op))
    return host(y).view(np.uint16)


@pytest.mark.parametrize("op,shape,nf,ns,parts,fold,split", CASES,
                         ids=[f"{c[5]}-{c[6]}" for c in CASES])
def test_folded_parts_give_the_bits_of_split_ones(op, shape, nf, ns, parts, fold, split):
    assert fg.kernel_name(desc(op, nf, shape), op) == "data_conv_" + fold
    assert fg.kernel_name(desc(op, ns, shape), op) == "data_conv_" + split
    assert parts_of_split(op, nf, shape) == 0 and parts_of_split(op, ns, shape) == parts
    x, W = _inputs(op, max(nf, ns), shape)
    both = min(nf, ns)
    np.testing.assert_array_equal(_run(op, nf, shape, x, W)[:both],
                                  _run(op, ns, shape, x, W)[:both])


def test_another_number_of_parts_gives_other_bits():
    shape, n, m = (29, 18, 320, 368, 3, 1, 1), 3, 1
    a, b = parts_of_split(FWD, n, shape), parts_of_split(FWD, m, shape)
    assert a and b and a != b, (a, b)
    x, W = _inputs(FWD, n, shape)
    assert (_run(FWD, n, shape, x, W)[:m] != _run(FWD, m, shape, x, W)).any()

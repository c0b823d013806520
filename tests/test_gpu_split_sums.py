"""The ordered sum of a kernel gradient's split partials, at part counts that
leave 0 to 3 parts over after the sum's groups of four loads: in one thread's
serial sum (up to 16 parts) and in each of 16 lanes (more). Inputs are -1, 0
and 1, so every partial and every sum is a whole number that fp16 holds and
the result is exact."""
import numpy as np
import pytest

import oracle
import paper_1909_11150_amd as fg
from gpu_util import dev, empty16, host, sample_indices, workspace

pytestmark = pytest.mark.gpu

# (n, h, w, c, k, r): parts
CASES = [
    ((3, 9, 41, 136, 136, 3), 3),
    ((2, 9, 41, 8, 8, 1), 4),
    ((3, 13, 100, 256, 256, 3), 7),
    ((3, 24, 41, 136, 136, 3), 8),
    ((2, 128, 100, 256, 256, 3), 14),
    ((1, 90, 20, 64, 64, 3), 15),
    ((2, 24, 41, 64, 64, 3), 16),
    ((1, 50, 41, 64, 64, 3), 17),      # one lane with two parts
    ((3, 50, 41, 16, 16, 3), 49),      # one lane with four, the rest three
    ((2, 40, 100, 16, 16, 3), 63),
    ((1, 128, 64, 16, 16, 3), 128),
    ((2, 90, 100, 8, 8, 1), 141),
]


@pytest.mark.parametrize("shape,parts", CASES, ids=[str(p) for _, p in CASES])
def test_sums_of_parts_are_exact(shape, parts):
    n, h, w, c, k, r = shape
    d = fg.ConvDesc.make(n, h, w, c, k, r, r, 1, r // 2)
    assert fg.workspace_bytes(d, fg.OP_BWD_WEIGHT) == 4 * parts * k * r * r * c
    rng = np.random.default_rng(parts)
    x = rng.integers(-1, 2, (n, h, w, c)).astype(np.float16)
    dy = rng.integers(-1, 2, (n, h, w, k)).astype(np.float16)
    dw = empty16((k, r, r, c))
    fg.conv2d_bwd_weight(d, dev(x), dev(dy), dw, workspace(d, fg.OP_BWD_WEIGHT))
    idx = sample_indices((k, r, r, c), 2500, rng)
    ref = oracle.conv2d_bwd_weight_points(x, dy, r, r, idx, 1, r // 2)
    assert np.abs(ref).max() <= 2048
    np.testing.assert_array_equal(host(dw).ravel()[idx].astype(np.float64), ref)

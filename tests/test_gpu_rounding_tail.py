"""One rounding from fp64 to fp16 at and beside every tie, and the unscale
check's values after the last whole vector."""
import numpy as np
import pytest
import torch

import paper_1909_11150_amd as fg
from gpu_util import dev, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("scale", [1.0, 1.0 + 2.0 ** -40, 1.0 - 2.0 ** -40, 2.0 ** -14,
                                   2.0 ** -14 * (1 + 2.0 ** -45)])
def test_fp64_to_fp16_beside_ties(scale):
    """y = 0, t = minus the midpoint of every two neighbouring fp16 numbers:
    the product with the scale lies on a tie or 2^-40 of it to either side,
    which fp32 does not resolve."""
    h = np.arange(0x7C00, dtype=np.uint16).view(np.float16).astype(np.float64)
    up = np.append(h[1:], 65536.0)
    t = -((h + up) / 2).astype(np.float32)
    t = np.concatenate([t, -t])
    y = np.zeros(t.size, np.float16)
    dy = torch.empty(t.size, dtype=torch.float16, device="cuda")
    fg.l2_head_grad(dev(y), dev(t), scale, dy)
    with np.errstate(over="ignore"):
        want = (-t.astype(np.float64) * np.float64(scale)).astype(np.float16)
    np.testing.assert_array_equal(host(dy).view(np.uint16), want.view(np.uint16))


@pytest.mark.parametrize("n", [1, 7, 8, 9, 15, 4096 + 1, 2 * 4096 - 1, 4096 * 3 + 7])
@pytest.mark.parametrize("bad", [False, True])
def test_unscale_tail(n, bad):
    """Lengths around a vector and a workgroup; a non-finite last value raises
    the flag, and nothing past the end is written."""
    rng = np.random.default_rng(n)
    g = rng.normal(size=n).astype(np.float16)
    if bad:
        g[-1] = np.inf
    out = torch.full((n + 8,), 7.0, dtype=torch.float32, device="cuda")
    flag = torch.zeros(1, dtype=torch.int32, device="cuda")
    inv = np.float32(2.0 ** -10)
    fg.grad_unscale_check(dev(g), inv, out, flag, numel=n)
    got = host(out)
    np.testing.assert_array_equal(got[:n], g.astype(np.float32) * inv)
    assert np.all(got[n:] == 7.0) and int(host(flag)[0]) == int(bad)

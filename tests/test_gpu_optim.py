"""GPU parity of lars_adam_update (layer-wise adaptive Adam, Section 6.2)
against the fp64 oracle on the same fp32 inputs.

Layers of ragged sizes (one element, tails that are not a multiple of four,
several workgroups); moments, weights and gradients seeded. The GPU works in
fp32, so each moment must agree to a few roundings of its two terms
(which can cancel), and the applied step must be lr * tau * u recomputed in
fp64 from the stored moments (tau = ||w|| / ||u||, within 1e-4 of the
oracle's) to 1e-5 of its size plus one ulp of w; the fp16 working copy is
checked bit for bit against the nearest-even rounding of the GPU's own fp32
weights. The oracle takes the fp32 values of the hyperparameters, which are
what the kernel receives (fp32 0.999 differs from 0.999 by 1.3e-8, a 1.3e-5
relative change of 1 - beta2). A flagged step must change nothing; the step count advances only
on applied steps; repeated runs are bit-identical.
"""
import numpy as np
import pytest
import torch

import paper_1909_11150_amd as fg
from gpu_util import OPT_HP as HP, check_opt_layer

pytestmark = pytest.mark.gpu

SIZES = [1, 5, 4096, 4099, 100003, 262144 + 3]


def _state(seed, sizes=SIZES, wscale=0.05):
    rng = np.random.default_rng(seed)
    w = [(rng.normal(size=n) * wscale).astype(np.float32) for n in sizes]
    m = [(rng.normal(size=n) * 1e-4).astype(np.float32) for n in sizes]
    v = [(rng.random(n) * 1e-7).astype(np.float32) for n in sizes]
    g = [(rng.normal(size=n) * 10.0 ** rng.uniform(-5, -2)).astype(np.float32) for n in sizes]
    return w, m, v, g


class Dev:
    def __init__(self, w, m, v, g, step=0):
        t = lambda a: torch.from_numpy(a.copy()).cuda()
        self.w32, self.m, self.v, self.g = [t(a) for a in w], [t(a) for a in m], \
            [t(a) for a in v], [t(a) for a in g]
        self.w16 = [torch.empty(a.shape, dtype=torch.float16, device="cuda") for a in w]
        self.step = torch.tensor([step], dtype=torch.int32, device="cuda")
        self.tens = fg.opt_tensors(self.w32, self.w16, self.m, self.v, self.g)
        self.ws = torch.empty(max(16, fg.lars_adam_workspace_bytes(self.tens)),
                              dtype=torch.uint8, device="cuda")

    def update(self, lr, flags=None):
        fg.lars_adam_update(self.tens, lr, flags, self.step, self.ws, **HP)
        torch.cuda.synchronize()

    def host(self):
        c = lambda ts: [x.cpu().numpy() for x in ts]
        return c(self.w32), c(self.m), c(self.v), c(self.w16), int(self.step.item())


def test_update_matches_oracle():
    w, m, v, g = _state(1)
    d = Dev(w, m, v, g, step=6)
    lr = 2e-3
    d.update(lr)
    w1, m1, v1, h1, step = d.host()
    assert step == 7
    for i in range(len(SIZES)):
        check_opt_layer(w[i], m[i], v[i], g[i], 7, lr, w1[i], m1[i], v1[i], h1[i])


def test_three_steps_follow_the_oracle():
    w, m, v, g = _state(2, sizes=[4099, 70000])
    d = Dev(w, m, v, g)
    rng = np.random.default_rng(3)
    for t in (1, 2, 3):
        gs = [(rng.normal(size=x.size) * 1e-3).astype(np.float32) for x in w]
        for i, x in enumerate(gs):
            d.g[i].copy_(torch.from_numpy(x))
        w0, m0, v0, _, _ = d.host()
        d.update(1e-2)
        w1, m1, v1, h1, step = d.host()
        assert step == t
        for i in range(2):
            check_opt_layer(w0[i], m0[i], v0[i], gs[i], t, 1e-2, w1[i], m1[i], v1[i], h1[i])


def test_flagged_step_changes_nothing():
    w, m, v, g = _state(4)
    d = Dev(w, m, v, g, step=3)
    for i in range(len(SIZES)):
        d.w16[i].fill_(7.0)
    before = d.host()
    flags = torch.tensor([0, 0, 1, 0], dtype=torch.int32, device="cuda")
    d.update(1e-2, flags)
    after = d.host()
    for a, b in zip(before[:4], after[:4]):
        assert all(np.array_equal(x.view(np.uint8), y.view(np.uint8)) for x, y in zip(a, b))
    assert after[4] == 3
    d.update(1e-2, torch.zeros(4, dtype=torch.int32, device="cuda"))
    assert d.host()[4] == 4


def test_zero_weight_layer_and_determinism():
    sizes = [1000, 4096]
    w, m, v, g = _state(5, sizes=sizes)
    w[0][:] = 0.0
    outs = []
    for _ in range(2):
        d = Dev(w, m, v, g)
        d.update(1e-3)
        outs.append(d.host())
    for a, b in zip(outs[0][0], outs[1][0]):
        assert np.array_equal(a.view(np.uint32), b.view(np.uint32))
    w1, m1, v1, h1, _ = outs[0]
    check_opt_layer(w[0], m[0], v[0], g[0], 1, 1e-3, w1[0], m1[0], v1[0], h1[0])


def _split(d, lr, ranges, flags=None, fmt=fg.GRAD_F32, inv=1.0, g=None):
    """The update as norms over the given layer ranges, then the apply."""
    tens = d.tens if g is None else fg.opt_tensors(d.w32, d.w16, d.m, d.v, g)
    for first, count in ranges:
        fg.lars_adam_norms(tens, first, count, d.step, d.ws, fmt, inv, **HP)
    fg.lars_adam_apply(tens, lr, flags, d.step, d.ws, fmt, inv, **HP)
    torch.cuda.synchronize()


def _bits_equal(a, b):
    return all(np.array_equal(x.view(np.uint8), y.view(np.uint8))
               for xs, ys in zip(a[:4], b[:4]) for x, y in zip(xs, ys)) and a[4] == b[4]


def test_split_update_equals_update():
    """Norms per range of layers (any split) then apply: the same bits as
    lars_adam_update."""
    w, m, v, g = _state(6)
    ref = Dev(w, m, v, g, step=2)
    ref.update(3e-3)
    for ranges in ([(0, len(SIZES))], [(3, 3), (0, 1), (1, 2)],
                   [(i, 1) for i in reversed(range(len(SIZES)))]):
        d = Dev(w, m, v, g, step=2)
        _split(d, 3e-3, ranges)
        assert _bits_equal(d.host(), ref.host()), ranges


def test_fp16_scaled_gradients_equal_unscaled_fp32():
    """The optimizer reading fp16 loss-scaled gradients with 1/S gives the
    bits it gives on the fp32 gradients the unscale check writes for them."""
    sizes = [3, 4096, 70001, 262147]
    w, m, v, _ = _state(7, sizes)
    rng = np.random.default_rng(8)
    S = 2.0 ** 13
    g16 = [(rng.normal(size=n) * 1e-3 * S).astype(np.float16) for n in sizes]
    g32 = [x.astype(np.float32) * np.float32(1.0 / S) for x in g16]
    a = Dev(w, m, v, g32, step=4)
    a.update(1e-3)
    b = Dev(w, m, v, g32, step=4)
    gd = [torch.from_numpy(x).cuda() for x in g16]
    _split(b, 1e-3, [(2, 2), (0, 2)], fmt=fg.GRAD_F16_SCALED, inv=1.0 / S, g=gd)
    assert _bits_equal(a.host(), b.host())
    w1, m1, v1, h1, _ = b.host()
    for i in range(len(sizes)):
        check_opt_layer(w[i], m[i], v[i], g32[i], 5, 1e-3, w1[i], m1[i], v1[i], h1[i])


def test_apply_needs_norms_of_every_layer():
    w, m, v, g = _state(9, [100, 5000, 17])
    d = Dev(w, m, v, g)
    before = d.host()
    fg.lars_adam_norms(d.tens, 0, 2, d.step, d.ws, **HP)
    with pytest.raises(fg.FgError):      # layer 2 not covered
        fg.lars_adam_apply(d.tens, 1e-3, None, d.step, d.ws, **HP)
    fg.lars_adam_norms(d.tens, 2, 1, d.step, d.ws, fg.GRAD_F16_SCALED, 0.5, **HP)
    with pytest.raises(fg.FgError):      # another gradient form: coverage restarts
        fg.lars_adam_apply(d.tens, 1e-3, None, d.step, d.ws, **HP)
    torch.cuda.synchronize()
    assert _bits_equal(d.host(), before)
    _split(d, 1e-3, [(1, 2), (0, 1)])
    assert d.host()[4] == 1
    with pytest.raises(fg.FgError):      # consumed by the apply
        fg.lars_adam_apply(d.tens, 1e-3, None, d.step, d.ws, **HP)


@pytest.mark.parametrize("grad", ["fp32", "fp16"])
def test_update_beyond_the_cache_keeps_the_bits(grad):
    """A layer's update does not depend on the others: with a layer added that
    takes the arrays past the Infinity Cache (256 MiB of reads, where the norms
    pass reads non-temporally), the small layers keep every bit; the large
    layer's first moments and fp16 copies follow the update rule."""
    big = (256 << 20) // (16 if grad == "fp32" else 14) + 1
    w, m, v, g = _state(10)
    if grad == "fp16":
        g = [(x * 2.0 ** 10).astype(np.float16) for x in g]
    inv = 2.0 ** -10 if grad == "fp16" else 1.0
    fmt = fg.GRAD_F16_SCALED if grad == "fp16" else fg.GRAD_F32
    outs = []
    for extra in (0, big):
        d = Dev(w, m, v, [x.astype(np.float32) for x in g], step=6)
        ts = [list(x) for x in (d.w32, d.w16, d.m, d.v,
                                [torch.from_numpy(x.copy()).cuda() for x in g])]
        if extra:
            gen = torch.Generator(device="cuda").manual_seed(3)
            one = lambda s: torch.randn(extra, device="cuda", generator=gen) * s
            for t, x in zip(ts, (one(0.05), torch.empty(extra, dtype=torch.float16,
                                                        device="cuda"),
                                 one(1e-4), one(1e-4).square_(),
                                 one(1e-3 / inv).to(ts[4][0].dtype))):
                t.append(x)
            before = [t[-1][:4096].cpu().numpy() for t in ts]
        tens = fg.opt_tensors(*ts)
        ws = torch.empty(fg.lars_adam_workspace_bytes(tens), dtype=torch.uint8, device="cuda")
        n = len(ts[0])
        fg.lars_adam_norms(tens, 0, n, d.step, ws, fmt, inv, **HP)
        fg.lars_adam_apply(tens, 2e-3, None, d.step, ws, fmt, inv, **HP)
        torch.cuda.synchronize()
        outs.append(d.host())
    assert _bits_equal(outs[0], outs[1])
    w1, m1, v1, h1, _ = outs[1]
    for i in range(len(SIZES)):
        gi = g[i].astype(np.float32) * np.float32(inv)
        check_opt_layer(w[i], m[i], v[i], gi, 7, 2e-3, w1[i], m1[i], v1[i], h1[i])
    # the large layer's moments and fp16 copy (its tau is a sum over all of it)
    w0, _, m0, v0, g0 = before
    gt = g0.astype(np.float32) * np.float32(inv)
    gt = gt.astype(np.float64) + np.float32(HP["weight_decay"]).astype(np.float64) * w0
    b1, b2 = (float(np.float32(HP[k])) for k in ("beta1", "beta2"))
    mb, vb = b1 * m0 + (1 - b1) * gt, b2 * v0 + (1 - b2) * gt * gt
    got = [t[-1][:4096].cpu().numpy() for t in ts]
    # a few fp32 roundings of each term, which may cancel
    assert np.all(np.abs(got[2] - mb) <= 2.0 ** -21 * (np.abs(m0) + np.abs(gt)))
    assert np.all(np.abs(got[3] - vb) <= 2.0 ** -21 * (v0 + gt * gt))
    assert np.array_equal(got[1].view(np.uint16), got[0].astype(np.float16).view(np.uint16))

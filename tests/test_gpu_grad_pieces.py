"""Pack and unpack on both sides of the lines between their two piece searches (16
pieces for pack, 2 for unpack; pack's gaps count), and with a full table: every
bit against the host's copies."""
import numpy as np
import pytest
import torch

import paper_1909_11150_amd as fg
from gpu_util import dev, host

pytestmark = pytest.mark.gpu

# members, whether each is followed by a gap (a piece of its own for pack)
CASES = [(1, False), (2, False), (3, False), (15, False), (16, False), (17, False),
         (1, True), (8, True), (9, True), (63, False), (64, False), (64, True)]


@pytest.mark.parametrize("members,gaps", CASES, ids=str)
def test_every_piece_is_found(members, gaps):
    rng = np.random.default_rng(members * 2 + gaps)
    # some of one workgroup or less, some of several, each end inside a workgroup
    sizes = [int(8 * rng.integers(1, 4000)) - (3 if gaps else 0) for _ in range(members)]
    off = np.cumsum([0] + [(n + 7) // 8 * 8 for n in sizes])
    total = int(off[-1])
    off = [int(o) for o in off[:-1]]
    src = [rng.integers(0, 1 << 16, n, dtype=np.uint16) for n in sizes]
    want = np.zeros(total, np.uint16)
    for o, s in zip(off, src):
        want[o:o + s.size] = s
    g16 = torch.full((total,), 7.0, dtype=torch.float16, device="cuda")
    fg.grad_group_pack([dev(s.view(np.float16)) for s in src], off, g16)
    np.testing.assert_array_equal(host(g16).view(np.uint16), want)

    g32 = rng.integers(0, 1 << 32, total, dtype=np.uint32)
    dst = [torch.full((n,), 7.0, device="cuda") for n in sizes]
    fg.grad_group_unpack(torch.from_numpy(g32.view(np.float32)).cuda(), dst, off)
    for o, d in zip(off, dst):
        np.testing.assert_array_equal(host(d).view(np.uint32), g32[o:o + d.numel()])

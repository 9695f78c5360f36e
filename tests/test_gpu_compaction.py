"""GPU test of the compaction of group flags on either side of the size at which the
blocks' counts are scanned by a launch of their own (2048 blocks of 2048 flags): the groups
cover all particles, and a partial walk, whose list and order come from the same kernels,
evaluates exactly the groups that hold an active particle."""

import numpy as np
import pytest

from gpu_helpers import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [2048 * 2048, 2048 * 2048 + 1, 2048 * 2049 + 1])
def test_groups_and_partial_walk(n):
    import torch
    import paper_1106_1900_amd as bh
    say("case compaction", n)
    g = torch.Generator(device="cuda")
    g.manual_seed(17)
    pos = torch.rand(n, 3, generator=g, device="cuda", dtype=torch.float64)
    mass = torch.full((n,), 1.0 / n, device="cuda", dtype=torch.float64)
    active = (torch.rand(n, generator=g, device="cuda") < 2e-4).to(torch.uint8)
    active[0] = active[n - 1] = 1
    with bh.Context() as ctx:
        ctx.build_tree(pos, mass)
        one = [x.clone() for x in ctx.compute_forces(1.0, 0.01)]
        two = [x.clone() for x in ctx.compute_forces(1.0, 0.02)]
        ctx.compute_forces(1.0, 0.01, want=False)
        got = ctx.compute_forces_active(1.0, 0.02, active)
        ex = ctx.export_tree()
    first, count = ex["gfirst"].astype(np.int64), ex["gcount"].astype(np.int64)
    assert first[0] == 0 and np.array_equal(first[1:], np.cumsum(count)[:-1])
    assert count.sum() == n and count.min() >= 1 and count.max() <= 64
    held = active.cpu().numpy()[ex["perm"]].astype(np.int64)        # in sorted order
    walked = np.repeat(np.add.reduceat(held, first) > 0, count)
    sel = np.empty(n, bool)
    sel[ex["perm"]] = walked
    sel = torch.from_numpy(sel).cuda()
    assert 100 < int(active.sum()) and not bool(sel.all())
    for x, a, b in zip(got, one, two):
        w = sel if x.dim() == 1 else sel[:, None]
        assert torch.equal(x, torch.where(w, b, a))

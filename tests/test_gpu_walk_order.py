"""GPU tests of the order of the groups on either side of the counts at which the small size
classes share a place in it (8 and 24 groups per wavefront; one cluster and many): a walk
evaluates every particle, with the bits of walks of half of the groups, which are ordered
by another rule."""

import pytest

from gpu_helpers import say

pytestmark = pytest.mark.gpu


def _system(n):
    """Radii over several decades: groups of all sizes."""
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    r = torch.rand(n, 1, generator=g, device="cuda", dtype=torch.float64) ** 1.5
    d = torch.randn(n, 3, generator=g, device="cuda", dtype=torch.float64)
    pos = (r * d / d.norm(dim=1, keepdim=True)).contiguous()
    return pos, torch.full((n,), 1.0 / n, device="cuda", dtype=torch.float64)


def _per_wave(ctx):
    import torch
    return ctx.stats().as_dict()["ngroups"] / (
        16 * torch.cuda.get_device_properties(0).multi_processor_count)


@pytest.mark.parametrize("n,lo,hi", [
    (150_000, 1, 4), (400_000, 4, 8), (800_000, 8, 24), (2_400_000, 24, 60),
])
def test_every_group_is_walked(n, lo, hi):
    import torch
    import paper_1106_1900_amd as bh
    say("case walk order", n)
    pos, mass = _system(n)
    with bh.Context() as ctx:
        ctx.build_tree(pos, mass)
        ctx.compute_forces(0.9, 0.01, want=False)
        full = [x.clone() for x in ctx.compute_forces(0.9, 0.02)]
        assert lo < _per_wave(ctx) <= hi
        for half in (pos[:, 0] < 0, pos[:, 0] >= 0):
            ctx.compute_forces(0.9, 0.01, want=False)
            got = ctx.compute_forces_active(0.9, 0.02, half.to(torch.uint8).contiguous())
            for x, y in zip(got, full):
                assert torch.equal(x[half], y[half])


def test_every_group_of_many_clusters():
    import torch
    import paper_1106_1900_amd as bh
    say("case walk order, 200 clusters")
    n, clusters = 800_000, 200
    pos, mass = _system(n)

    def forces(lo, hi):
        one = dict(n=n // clusters, theta=0.75, dt=1e-3)
        part = slice(lo * (n // clusters), hi * (n // clusters))
        with bh.Context() as ctx:
            ctx.batch_build([dict(one, eps=0.01)] * (hi - lo), pos[part], mass[part])
            ctx.batch_forces(want=False)
            ctx.batch_set_params([dict(one, eps=0.02)] * (hi - lo))
            return [x.clone() for x in ctx.batch_forces()], _per_wave(ctx)

    full, per_wave = forces(0, clusters)
    halves = [forces(0, 100), forces(100, 200)]
    assert 8 < per_wave <= 24 and all(p <= 8 for _, p in halves)
    for k in range(2):
        assert torch.equal(full[k], torch.cat([h[k] for h, _ in halves]))

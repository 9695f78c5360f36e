"""GPU tests of the walk's hand-out where some groups are left to single wavefronts: small
clusters beside larger ones, groups of up to 16 particles, and more groups than
wavefronts in wide workgroups; forces and counts against the oracle."""

import numpy as np
import pytest

import oracle
import workloads
from gpu_helpers import compare_forces, say, to_dev

pytestmark = pytest.mark.gpu

THETA, EPS = 0.6, 0.01


@pytest.mark.parametrize("sizes,ncrit", [
    ((320, 321, 64, 1, 2, 700), 64),        # either side of the small clusters' line
    ((16,) * 200 + (3000,), 64),            # few groups of a larger one behind many small
    ((4096,), 16),                          # no group large enough for a team
    ((2500, 17, 5000), 20),
    ((8100,), 1),                           # twice as many groups as wavefronts
])
def test_batches_of_small_clusters_and_groups(sizes, ncrit):
    import paper_1106_1900_amd as bh
    say("case handout", sizes[-1], len(sizes), ncrit)
    leaf = min(16, ncrit)
    parts = [workloads.plummer(n, 50 + i) for i, n in enumerate(sizes)]
    pos = np.concatenate([p for p, _, _ in parts])
    mass = np.concatenate([m for _, _, m in parts])
    clusters = [dict(n=n, theta=THETA, eps=EPS, nleaf=leaf, ncrit=ncrit) for n in sizes]
    active = np.zeros(len(mass), np.uint8)
    active[::3] = 1
    with bh.Context() as ctx:
        ctx.batch_build(clusters, to_dev(pos), to_dev(mass))
        acc, pot = (x.cpu().numpy() for x in ctx.batch_forces())
        ex = ctx.export_tree()
        a2, p2 = ctx.compute_forces_active(THETA, EPS, to_dev(active))
        assert np.array_equal(a2.cpu().numpy(), acc) and np.array_equal(p2.cpu().numpy(), pot)
    first, g0 = 0, 0
    for n, (p, _, m) in zip(sizes, parts):
        t = oracle.Tree(p, m, leaf, ncrit)
        npp, npc = t.walk_counts(THETA)
        assert np.array_equal(ex["npp"][g0:g0 + t.ngroups], npp)
        assert np.array_equal(ex["npc"][g0:g0 + t.ngroups], npc)
        g0 += t.ngroups
        groups = np.linspace(0, t.ngroups - 1, min(t.ngroups, 24)).astype(np.int64)
        if n > 1 and n != 16:
            compare_forces(acc[first:first + n], pot[first:first + n], t, THETA, EPS, groups=groups)
        first += n

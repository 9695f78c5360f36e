"""GPU tests of the moments where the leaf size decides how they are split: runs of one, two
and four tiles, on either side of the sizes where that changes, runs with more cells than
fit on chip, systems that one workgroup holds or just does not, clusters smaller than
their leaves, and the workgroups of large systems; builds and refits against the oracle."""

import numpy as np
import pytest

import oracle
import workloads
from gpu_helpers import compare_tree, compare_walk, gpu_build, say, to_dev

pytestmark = pytest.mark.gpu

THETA = 0.8


@pytest.mark.parametrize("n,nleaf", [
    (293, 1), (294, 1), (852, 1), (853, 1), (881, 8), (882, 8), (1025, 8), (2556, 8), (2560, 8), (4096, 13),
    (131_072, 3), (131_073, 2), (131_073, 3), (131_073, 13), (1 << 19, 5), ((1 << 19) + 1, 5),
    ((1 << 19) + 1, 13), ((1 << 21) + 1, 14),
])
def test_build_and_refit(n, nleaf):
    say("case moments leaves", n, nleaf)
    pos, vel, mass = workloads.plummer(n, 63)
    with gpu_build(pos, mass, nleaf, 64) as ctx:
        ctx.set_velocities(to_dev(vel))
        ctx.compute_forces(THETA, 0.01, want=False)
        t = oracle.Tree(pos, mass, nleaf, 64)
        ex = ctx.export_tree()
        compare_tree(ex, t)
        ctx.drift(1 / 64)
        ctx.refit()
        ctx.compute_forces(THETA, 0.01, want=False)
        t.refit(pos + vel * (1 / 64))
        ex = ctx.export_tree()
        compare_tree(ex, t)
        if n < 200_000:
            compare_walk(ex, t, THETA)


@pytest.mark.parametrize("sizes,nleaf", [((2,) * 1100, 16), ((1, 3, 2, 5) * 400, 16),
                                         ((2,) * 300 + (3000,), 4), ((2,) * 70_000, 64)])
def test_clusters_smaller_than_their_leaves(sizes, nleaf):
    import paper_1106_1900_amd as bh
    say("case moments of tiny clusters", len(sizes), nleaf)
    n = sum(sizes)
    rng = np.random.default_rng(18)
    pos, vel = rng.normal(0.0, 1.0, (n, 3)), rng.normal(0.0, 1.0, (n, 3))
    mass = rng.uniform(0.5, 1.5, n) / n
    clusters = [dict(n=s, theta=THETA, eps=0.01, nleaf=nleaf, ncrit=64) for s in sizes]
    some = sorted({0, 1, 7, len(sizes) // 2, len(sizes) - 2, len(sizes) - 1})
    first = np.concatenate([[0], np.cumsum(sizes)])
    with bh.Context() as ctx:
        ctx.batch_build(clusters, to_dev(pos), to_dev(mass), to_dev(vel))
        ctx.batch_forces(want=False)
        ex = ctx.export_tree()
        roots = {c: ex["com"][c].copy() for c in some}      # the roots come first
        assert np.array_equal(ex["mass"][some],
                              [oracle.Tree(pos[first[c]:first[c + 1]], mass[first[c]:first[c + 1]],
                                           nleaf, 64).moments()["mass"][0] for c in some])
        ctx.drift(0.25)
        ctx.refit()
        ex2 = ctx.export_tree()
    for c in some:
        s = slice(first[c], first[c + 1])
        t = oracle.Tree(pos[s], mass[s], nleaf, 64)
        assert np.array_equal(roots[c], t.moments()["com"][0])
        t.refit(pos[s] + vel[s] * 0.25)
        assert np.array_equal(ex2["com"][c], t.moments()["com"][0])

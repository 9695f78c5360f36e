"""GPU tests of the walk's hand-out: a group walked by a whole workgroup (few groups)
gives the bits that a wavefront alone gives (the same cluster inside a batch with
many groups), whatever its size class and lane mode, and both match the oracle."""

import numpy as np
import pytest

import oracle
import workloads
from gpu_helpers import compare_forces, compare_walk, say, to_dev

pytestmark = pytest.mark.gpu

# n, nleaf, ncrit: one group; few groups (workgroups of eight wavefronts, all groups
# walked by teams); more than a quarter of the grid's wavefronts (large groups only);
# groups of 65 to 128 particles with two or three particles per lane
CASES = [(1, 16, 64), (3, 16, 64), (64, 16, 64), (128, 64, 128), (130, 16, 128), (1500, 16, 64),
         (4096, 8, 26), (8192, 32, 128), (8193, 16, 64), (30000, 16, 64), (20011, 64, 128)]


@pytest.fixture(scope="module")
def crowd():
    """A companion of many groups, so that a batch with it walks group by group."""
    pos, _, mass = workloads.uniform_cube(200000, 5)
    return pos, mass, dict(n=200000, theta=0.9, eps=0.01, nleaf=8, ncrit=8)


@pytest.mark.parametrize("n,nleaf,ncrit", CASES)
def test_team_walk_equals_single_walk(crowd, n, nleaf, ncrit):
    import paper_1106_1900_amd as bh
    say("case", n, nleaf, ncrit)
    pos, _, mass = workloads.plummer(n, 31)
    theta, eps = 0.6, 0.01
    one = bh.Context(nleaf=nleaf, ncrit=ncrit)
    one.build_tree(to_dev(pos), to_dev(mass))
    a1, p1 = one.compute_forces(theta, eps)
    a1, p1 = a1.cpu().numpy(), p1.cpu().numpy()
    t = oracle.Tree(pos, mass, nleaf, ncrit)
    ex = one.export_tree()
    compare_walk(ex, t, theta)
    if n > 1:
        groups = np.linspace(0, t.ngroups - 1, min(t.ngroups, 64)).astype(np.int64)
        compare_forces(a1, p1, t, theta, eps, groups=groups)
    # only some groups: those of an active particle in every seventh
    mask = np.zeros(n, np.uint8)
    mask[ex["perm"][ex["gfirst"][::7]]] = 1
    a2, p2 = one.compute_forces_active(theta, eps, to_dev(mask))
    assert np.array_equal(a2.cpu().numpy(), a1) and np.array_equal(p2.cpu().numpy(), p1)
    one.close()
    # the same cluster between the groups of a large one
    cpos, cmass, cprm = crowd
    clusters = [dict(n=n, theta=theta, eps=eps, nleaf=nleaf, ncrit=ncrit), cprm]
    with bh.Context() as ctx:
        ctx.batch_build(clusters, to_dev(np.concatenate([pos, cpos])),
                        to_dev(np.concatenate([mass, cmass])))
        a, p = ctx.batch_forces()
        assert ctx.stats().ngroups > 4 * 4096
        assert np.array_equal(a.cpu().numpy()[:n], a1) and np.array_equal(p.cpu().numpy()[:n], p1)

"""GPU tests of the moments' split into runs of about 1024 particles and units of runs:
trees at the sizes where a run, a workgroup's runs or the number of launches change, trees
with more cells in a run than it holds on chip, leaves longer than a run, cells across
clusters' starts, and refits of them, against the oracle."""

import numpy as np
import pytest

import oracle
import workloads
from gpu_helpers import compare_tree, compare_walk, gpu_build, say, to_dev

pytestmark = pytest.mark.gpu


def _plummer(n):
    return workloads.plummer(n, 61)


def _coincident(n):
    # a leaf of 2700 coincident particles (it covers whole runs) in a cluster
    pos, vel, mass = workloads.plummer(n, 62)
    sel = np.random.default_rng(8).permutation(n)[:2700]
    pos[sel] = pos[sel[0]]
    return pos, vel, mass


# name: particles, leaf size
CASES = {
    "n1023": (_plummer, 1023, 16), "n1024": (_plummer, 1024, 16), "n1025": (_plummer, 1025, 16),
    "n4096": (_plummer, 4096, 16), "n4097": (_plummer, 4097, 16), "n5120": (_plummer, 5120, 7),
    "n4096_leaf1": (_plummer, 4096, 1), "n6000_leaf1": (_plummer, 6000, 1),
    "n6000_leaf64": (_plummer, 6000, 64), "n3500_coincident": (_coincident, 3500, 16),
    "n9000_coincident": (_coincident, 9000, 16),
    "n262144": (_plummer, 1 << 18, 16), "n262145": (_plummer, (1 << 18) + 1, 16),
    "n524288": (_plummer, 1 << 19, 16), "n524289": (_plummer, (1 << 19) + 1, 16),
    "n600001_leaf2": (_plummer, 600_001, 2),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_build_and_refit(name):
    make, n, nleaf = CASES[name]
    pos, vel, mass = make(n)
    theta = 0.7
    say("case moments", name)
    with gpu_build(pos, mass, nleaf, 64) as ctx:
        ctx.set_velocities(to_dev(vel))
        ctx.compute_forces(theta, 0.01, want=False)
        t = oracle.Tree(pos, mass, nleaf, 64)
        ex = ctx.export_tree()
        compare_tree(ex, t)
        compare_walk(ex, t, theta)
        ctx.drift(1 / 64)
        ctx.refit()
        ctx.compute_forces(theta, 0.01, want=False)
        t.refit(pos + vel * (1 / 64))
        ex = ctx.export_tree()
        compare_tree(ex, t)
        compare_walk(ex, t, theta)


def _check_nodes(ex):
    # a node's mass and centre of mass are its children's in array order, bit for bit
    node = np.nonzero(ex["is_leaf"] == 0)[0]
    child, nchild = ex["child"][node], ex["nchild"][node]
    m, s = np.zeros(len(node)), np.zeros((len(node), 3))
    for k in range(8):
        has = nchild > k
        c = child[has] + k
        m[has] += ex["mass"][c]
        s[has] += ex["mass"][c][:, None] * ex["com"][c]
    assert np.array_equal(ex["mass"][node], m)
    assert np.array_equal(ex["com"][node], s / m[:, None])


def test_nodes_of_clusters_and_of_the_largest_split():
    import paper_1106_1900_amd as bh
    # clusters shorter and longer than a run and than 64 runs, in more than 512 runs
    sizes = [1, 700, 1024, 1, 90_000, 3, 5000, 150_001, 2048, 400_000]
    parts = [workloads.plummer(n, 70 + i) for i, n in enumerate(sizes)]
    say("case moments of a batch", sizes)
    with bh.Context() as ctx:
        ctx.batch_build([dict(n=n, theta=0.75, eps=0.01) for n in sizes],
                        to_dev(np.concatenate([p for p, _, _ in parts])),
                        to_dev(np.concatenate([m for _, _, m in parts])))
        _check_nodes(ctx.export_tree())
    # more than 512 units of 64 runs
    n = (1 << 25) + 70_000
    say("case moments", n)
    rng = np.random.default_rng(9)
    pos, mass = rng.standard_normal((n, 3)), rng.random(n) + 0.5
    with bh.Context(nleaf=64) as ctx:
        ctx.build_tree(to_dev(pos), to_dev(mass))
        _check_nodes(ctx.export_tree())

"""GPU tests of the sizes at which a build has fewer launches: up to 16 tiles of 256
particles the cells' kernel scans the level counts, up to four blocks of 2048 flags the
compaction counts them, and up to 1024 chunks of 4096 particles a cluster's cube is made
with its keys.  Trees, groups and lists of active groups equal the oracle's bit for bit on
both sides of each line."""

import numpy as np
import pytest

import oracle
import workloads
from gpu_helpers import compare_tree, compare_walk, gpu_build, say, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 2, 255, 257, 2048, 2049, 4096, 4097, 8192, 8193,
                               1024 * 4096, 1024 * 4096 + 1])
def test_build_at_the_lines(n):
    say("case launches", n)
    pos, _, mass = workloads.plummer(n, 91) if n > 1 else workloads.uniform_cube(1, 91)
    theta = 0.9
    with gpu_build(pos, mass) as ctx:
        t = oracle.Tree(pos, mass)
        if n > 10_000:
            compare_tree(ctx.export_tree(), t)
            return
        acc, pot = ctx.compute_forces(theta, 0.01)
        acc, pot = acc.cpu().numpy(), pot.cpu().numpy()
        ex = ctx.export_tree()
        compare_tree(ex, t)
        compare_walk(ex, t, theta)
        # one particle of every fifth group active: their groups' forces, and only those
        mask = np.zeros(n, np.uint8)
        mask[ex["perm"][ex["gfirst"][::5]]] = 1
        walked = np.zeros(n, bool)
        for f, c in zip(ex["gfirst"][::5], ex["gcount"][::5]):
            walked[ex["perm"][f:f + c]] = True
        a, p = ctx.compute_forces_active(theta, 0.01, to_dev(mask))
        a, p = a.cpu().numpy(), p.cpu().numpy()
        assert np.array_equal(a[walked], acc[walked]) and np.array_equal(p[walked], pot[walked])

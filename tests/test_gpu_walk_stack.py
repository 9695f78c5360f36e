"""GPU tests of the walk's stack of pending cells: opening angles at which it outgrows its
part in LDS (entries go to device memory and come back) and, with most cells opened, fills
so far that fewer cells are popped at a time; counts and forces against the oracle, by
single wavefronts and by whole workgroups."""

import numpy as np
import pytest

import oracle
import workloads
from gpu_helpers import compare_forces, compare_walk, gpu_build, host_threads, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("model,n,nleaf,ncrit,theta", [
    ("uniform_cube", 20_000, 1, 64, 0.1),       # nearly every cell opened, eight children each
    ("uniform_cube", 3_000, 1, 16, 0.1),        # whole workgroups walk the groups
    ("plummer", 60_000, 4, 32, 0.25),           # a deep tree
    ("clustered", 40_000, 8, 64, 0.15),
])
def test_deep_stacks(model, n, nleaf, ncrit, theta):
    say("case stack", model, n, nleaf, ncrit, theta)
    pos, _, mass = getattr(workloads, model)(n, 81)
    with gpu_build(pos, mass, nleaf, ncrit) as ctx:
        acc, pot = ctx.compute_forces(theta, 0.01)
        t = oracle.Tree(pos, mass, nleaf, ncrit)
        compare_walk(ctx.export_tree(), t, theta)
        groups = np.linspace(0, t.ngroups - 1, 48).astype(np.int64)
        compare_forces(acc.cpu().numpy(), pot.cpu().numpy(), t, theta, 0.01, groups=groups,
                       threads=host_threads())

"""GPU test of the rows of positions, velocities, accelerations and potentials in caller
order, at sizes around the blocks and the eight parts that the kernels go over: what was
loaded comes back bit for bit, each alone and together."""

import numpy as np
import pytest

import workloads
from gpu_helpers import gpu_build, say, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 3, 255, 256, 257, 2047, 2048, 2049, 30_001])
def test_rows_come_back(n):
    say("case rows", n)
    pos, vel, mass = workloads.uniform_cube(n, 17)
    vel = np.random.default_rng(n).standard_normal((n, 3))
    with gpu_build(pos, mass) as ctx:
        ctx.set_velocities(to_dev(vel))
        acc, pot = ctx.compute_forces(0.8, 0.02)
        x, v = ctx.get_positions()
        assert np.array_equal(x.cpu().numpy(), pos)
        assert np.array_equal(v.cpu().numpy(), vel)
        # a particle's acceleration follows it into any caller order
        perm = np.random.default_rng(5).permutation(n)
        with gpu_build(pos[perm], mass[perm]) as other:
            a, p = other.compute_forces(0.8, 0.02)
            assert np.array_equal(a.cpu().numpy(), acc.cpu().numpy()[perm])
            assert np.array_equal(p.cpu().numpy(), pot.cpu().numpy()[perm])

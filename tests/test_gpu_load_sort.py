"""GPU tests of the sort of a load and of batches (App. A: keys sorted with equal
keys in caller order) through buckets split at sampled keys: the order equals the
oracle's stable sort bit for bit for inputs whose order has a period (a lattice), that
are sorted already, that hold many coincident particles, and around the sizes at which
clusters get more buckets."""

import numpy as np
import pytest

import oracle
import workloads
from gpu_helpers import say, to_dev

pytestmark = pytest.mark.gpu


def _lattice():
    pos, _, mass = workloads.lattice(48)        # 110,592: stride and rows share factors
    return pos, mass


def _sorted():
    pos, _, mass = workloads.plummer(60_000, 3)
    perm, _ = oracle.Tree(pos, mass).order()
    return pos[perm[::-1]].copy(), mass


def _coincident():
    # one key held by 30,000 of 90,000 particles, another by 15,000
    pos, _, mass = workloads.plummer(90_000, 4)
    rng = np.random.default_rng(6)
    sel = rng.permutation(90_000)
    pos[sel[:30_000]] = pos[sel[0]]
    pos[sel[30_000:45_000]] = pos[sel[30_000]]
    return pos, mass


def _plummer(n):
    pos, _, mass = workloads.plummer(n, 7)
    return pos, mass


INPUTS = {
    "lattice": _lattice, "sorted": _sorted, "coincident": _coincident,
    "n4096": lambda: _plummer(4096), "n4097": lambda: _plummer(4097),
    "n8193": lambda: _plummer(8193), "n262144": lambda: _plummer(1 << 18),
    "n262145": lambda: _plummer((1 << 18) + 1), "n524289": lambda: _plummer((1 << 19) + 1),
}


def _check(ex, first, pos, mass):
    perm, key = oracle.Tree(pos, mass).order()
    n = len(mass)
    assert np.array_equal(ex["key"][first:first + n], key), "keys differ"
    assert np.array_equal(ex["perm"][first:first + n] - first, perm), "sorted order differs"


@pytest.mark.parametrize("name", sorted(INPUTS))
def test_load_order(name):
    import paper_1106_1900_amd as bh
    say("case load sort", name)
    pos, mass = INPUTS[name]()
    with bh.Context() as ctx:
        ctx.build_tree(to_dev(pos), to_dev(mass))
        _check(ctx.export_tree(), 0, pos, mass)


def test_batch_order_loaded_and_rebuilt():
    # clusters of one chunk and of several, with ties, in one batch; then rebuilt from
    # the held order with every cluster's positions permuted
    import paper_1106_1900_amd as bh
    parts = [_plummer(1), _coincident(), _plummer(4096), _plummer(5000), _lattice(), _plummer(2)]
    pos = np.concatenate([p for p, _ in parts])
    mass = np.concatenate([m for _, m in parts])
    say("case batch sort", [len(m) for _, m in parts])
    clusters = [dict(n=len(m), theta=0.75, eps=0.01) for _, m in parts]
    with bh.Context() as ctx:
        ctx.batch_build(clusters, to_dev(pos), to_dev(mass))
        ex = ctx.export_tree()
        rng = np.random.default_rng(9)
        first, new = 0, []
        for p, m in parts:
            _check(ex, first, p, m)
            new.append(p[rng.permutation(len(m))])
            first += len(m)
        ctx.set_state(to_dev(np.concatenate(new)), to_dev(np.zeros_like(pos)))
        ex = ctx.export_tree()
        first = 0
        for p, (_, m) in zip(new, parts):
            _check(ex, first, p, m)
            first += len(m)


@pytest.mark.parametrize("deep", [2, 16, 17, 40, 3000])
def test_pairs_that_agree_in_the_passes_window(deep):
    # `deep` particles in a cube of 2^-16 of the domain: their keys agree in the first
    # 48 bits, so the bucket's passes (40 bits below the first in which its keys
    # differ) leave them in arrival order and they are ordered afterwards, by one
    # thread or, when they are many, by passes over every bit; some coincide
    import paper_1106_1900_amd as bh
    n = 3500
    say("case window", deep)
    rng = np.random.default_rng(11)
    pos = rng.uniform(0.0, 1.0, (n, 3))
    pos[0], pos[1] = 0.0, 1.0
    sel = 2 + rng.permutation(n - 2)[:deep]
    pos[sel] = 0.3 + rng.uniform(0.0, 2.0 ** -17, (deep, 3))
    pos[sel[: deep // 2]] = pos[sel[0]]
    mass = np.full(n, 1.0 / n)
    with bh.Context() as ctx:
        ctx.build_tree(to_dev(pos), to_dev(mass))
        _check(ctx.export_tree(), 0, pos, mass)
        new = pos[rng.permutation(n)]
        ctx.set_state(to_dev(new), to_dev(np.zeros_like(pos)))
        _check(ctx.export_tree(), 0, new, mass)

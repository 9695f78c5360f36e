"""GPU tests of the bucket sort where its buckets are hard, for each of its three bucket
sizes (up to 2^18, 2^19 and 2^20 particles): many coincident particles (ties in caller
order, in LDS and in device memory), long runs of keys that agree in the passes' window,
and inputs whose sampled places say nothing about the rest, so that one bucket holds
nearly everything and is sorted through device memory.  The order of a load and of a
rebuild equals the oracle's stable sort bit for bit; so does that of batches of so many
tiny clusters that they take the radix sort."""

import numpy as np
import pytest

import oracle
import workloads
from gpu_helpers import say, to_dev

pytestmark = pytest.mark.gpu

# particles, buckets per chunk, pairs a bucket's LDS holds
SIZES = {"1024": (60_000, 4, 4096), "2048": (300_000, 2, 6144), "4096": (600_000, 1, 12288)}


def _check(ctx, pos, mass, first=0, ex=None):
    ex = ex or ctx.export_tree()
    perm, key = oracle.Tree(pos, mass).order()
    n = len(mass)
    assert np.array_equal(ex["key"][first:first + n], key), "keys differ"
    assert np.array_equal(ex["perm"][first:first + n] - first, perm), "sorted order differs"


def _load_and_rebuild(pos, mass):
    import paper_1106_1900_amd as bh
    with bh.Context() as ctx:
        ctx.build_tree(to_dev(pos), to_dev(mass))
        _check(ctx, pos, mass)
        new = pos[np.random.default_rng(3).permutation(len(mass))]
        ctx.set_state(to_dev(new), to_dev(np.zeros_like(new)))
        _check(ctx, new, mass)


@pytest.mark.parametrize("size", sorted(SIZES))
@pytest.mark.parametrize("share", [0.8, 1.2])
def test_coincident_below_and_above_the_lds_capacity(size, share):
    n, _, cap = SIZES[size]
    many = int(share * cap)
    say("case coincident", n, many)
    pos, _, mass = workloads.plummer(n, 12)
    sel = np.random.default_rng(13).permutation(n)
    pos[sel[:many]] = pos[sel[0]]                     # a bucket to itself
    pos[sel[many:many + 300]] = pos[sel[many]]        # a run within a bucket
    _load_and_rebuild(pos, mass)


@pytest.mark.parametrize("size", sorted(SIZES))
@pytest.mark.parametrize("close", [16, 18, 1500])
def test_keys_that_agree_in_the_passes_window(size, close):
    # a uniform cube, whose buckets' keys differ high up, and `close` particles within
    # 2^-18 of its side, half of them coincident
    n = SIZES[size][0]
    say("case window", n, close)
    rng = np.random.default_rng(14)
    pos = rng.uniform(0.0, 1.0, (n, 3))
    pos[0], pos[1] = 0.0, 1.0
    sel = 2 + rng.permutation(n - 2)[:close]
    pos[sel] = 0.3 + rng.uniform(0.0, 2.0 ** -18, (close, 3))
    pos[sel[: close // 2]] = pos[sel[0]]
    _load_and_rebuild(pos, np.full(n, 1.0 / n))


def _sampled(n, sub):
    """The places of a cluster's order whose keys the sort samples."""
    ncand = -(-n // 4096) * sub * 16
    stretch = n // ncand
    q = np.arange(ncand, dtype=np.uint64)
    at = (((q * 2654435761 & 0xffffffff) >> 16) * stretch) >> 16
    return (q * stretch + at).astype(np.int64)


@pytest.mark.parametrize("size", sorted(SIZES))
def test_samples_that_miss_nearly_all(size):
    # the sampled particles lie in a corner, all others in a cube apart: one bucket, of
    # distinct keys and some ties
    n, sub, _ = SIZES[size]
    say("case missed", n)
    rng = np.random.default_rng(15)
    dense = rng.uniform(0.4, 0.5, (n, 3))
    dense[::50] = dense[rng.integers(0, n // 40, len(dense[::50]))]
    corner = rng.uniform(0.9, 1.0, (n, 3))
    pos = dense.copy()
    pos[_sampled(n, sub)] = corner[_sampled(n, sub)]
    mass = np.full(n, 1.0 / n)
    import paper_1106_1900_amd as bh
    with bh.Context() as ctx:
        ctx.build_tree(to_dev(pos), to_dev(mass))
        ex = ctx.export_tree()
        _check(ctx, pos, mass, ex=ex)
        held = ex["perm"]                # a rebuild samples the held order
        new = dense.copy()
        new[held[_sampled(n, sub)]] = corner[held[_sampled(n, sub)]]
        ctx.set_state(to_dev(new), to_dev(np.zeros_like(new)))
        _check(ctx, new, mass)


def test_thousands_of_tiny_clusters():
    import paper_1106_1900_amd as bh
    k = 9000
    say("case tiny clusters", k)
    rng = np.random.default_rng(16)
    sizes = rng.integers(1, 30, k)
    sizes[7] = 5000
    n = int(sizes.sum())
    pos = rng.normal(0.0, 1.0, (n, 3))
    pos[rng.integers(0, n, n // 4)] = 0.25        # ties
    mass = np.full(n, 1.0 / n)
    clusters = [dict(n=int(s), theta=0.75, eps=0.01) for s in sizes]
    first = np.concatenate([[0], np.cumsum(sizes)])
    some = sorted({0, 1, 6, 7, 8, k - 1} | set(map(int, rng.integers(0, k, 100))))
    with bh.Context() as ctx:
        ctx.batch_build(clusters, to_dev(pos), to_dev(mass))
        ex = ctx.export_tree()
        for c in some:
            s = slice(first[c], first[c + 1])
            _check(ctx, pos[s], mass[s], first[c], ex)
        new = pos.copy()
        for c in some:
            s = slice(first[c], first[c + 1])
            new[s] = pos[s][rng.permutation(int(sizes[c]))]
        ctx.set_state(to_dev(new), to_dev(np.zeros_like(new)))
        ex = ctx.export_tree()
        for c in some:
            s = slice(first[c], first[c + 1])
            _check(ctx, new[s], mass[s], first[c], ex)

"""Hash-bucket layers whose states remember the generators that take them back:
sizes and exported layers against the sort path on the same calls. Every place
the bits can lie (above the key, in entry 0's place), sets of which all have a
bit, some, or none, repeated entries, involutions and pairs, layers that grow
and shrink between the one-workgroup kernel and the buckets. Exact."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from paper_2509_19162_amd import api  # noqa: E402
from paper_2509_19162_amd import inputs as I  # noqa: E402


def same(n, gens, **kw):
    got = api.growth_ex(n, gens, **kw)
    ref = api.growth_ex(n, gens, packed_sort=True, **kw)
    assert (got.status, got.sizes, got.states_expanded, got.candidates) == (
        ref.status, ref.sizes, ref.states_expanded, ref.candidates)
    if ref.layers is not None:
        assert len(got.layers) == len(ref.layers)
        for a, b in zip(got.layers, ref.layers):
            assert np.array_equal(a, b)


@pytest.mark.parametrize("n", [13, 14, 15, 16])
@pytest.mark.parametrize("fam", ["lrx", "coxeter", "pancake", "cyclic_coxeter", "star"])
def test_permutations(n, fam):
    gens = I.family(fam, n)
    start = [int(x) for x in I.rng_for(n, seed=5).permutation(n)]
    same(n, gens, start=start, max_layers=512, max_frontier=300_000, export_layers=2_000_000)


@pytest.mark.parametrize("n,counts", [(16, (8, 8)), (16, (4, 4, 4, 4)), (16, (7, 5, 2, 2)), (15, (5, 5, 5)),
                                      (14, (3, 3, 3, 3, 2)), (13, (4, 4, 5)), (12, (5, 5, 1, 1)), (11, (4, 4, 3))])
@pytest.mark.parametrize("fam", ["lrx", "coxeter"])
def test_repeated_entries(n, counts, fam):
    start = [c for c, m in enumerate(counts) for _ in range(m)]
    same(n, I.family(fam, n), start=start, max_layers=512, max_frontier=400_000, export_layers=2_000_000)


@pytest.mark.parametrize("n,ones,fam", [(24, 12, "lrx"), (32, 16, "lrx"), (60, 5, "lrx"), (61, 5, "lrx"),
                                        (62, 5, "lrx"), (64, 4, "lrx"), (28, 10, "coxeter"), (29, 10, "coxeter"),
                                        (30, 10, "coxeter"), (36, 7, "coxeter")])
def test_binary(n, ones, fam):
    start = [0] * (n - ones) + [1] * ones
    same(n, I.family(fam, n), start=start, binary_state=True, max_layers=512, max_frontier=400_000, export_layers=1_000_000)


@pytest.mark.parametrize("n,m,involutions", [(16, 1, 0), (16, 0, 2), (16, 1, 2), (16, 2, 0), (16, 2, 1), (13, 6, 0),
                                             (13, 6, 1), (14, 4, 0), (14, 3, 3), (15, 1, 1), (13, 8, 0), (13, 8, 1),
                                             (14, 6, 1), (15, 4, 1), (15, 8, 0), (15, 8, 1)])
def test_random_sets(n, m, involutions):
    r = I.rng_for(n, seed=91 + m)
    gens = I.random_perms_with_inverses(n, m, r) + [I.random_involution(n, r) for _ in range(involutions)]
    same(n, gens, max_layers=512 if len(gens) == 2 else 10, max_frontier=1_000_000)


@pytest.mark.parametrize("n", [14, 16])
def test_hand_over_to_the_sort_path(n, monkeypatch):
    kw = dict(max_layers=512, max_frontier=150_000, export_layers=1_000_000)
    ref = api.growth_ex(n, I.lrx(n), packed_sort=True, **kw)
    monkeypatch.setenv("CG_HASH_CANDIDATES", "100000")
    got = api.growth_ex(n, I.lrx(n), **kw)
    assert (got.status, got.sizes) == (ref.status, ref.sizes)
    for a, b in zip(got.layers, ref.layers):
        assert np.array_equal(a, b)

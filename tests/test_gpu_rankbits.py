"""Layers over a rank bitmap (permutations of up to 12 entries) against the
CPU oracle and, state by state, against the sort path: chains of small
steps, large steps by segments of the bitmap, steps from the side of the
unseen states, directed sets. Tolerance: none (exact integers)."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from paper_2509_19162_amd import api  # noqa: E402
from paper_2509_19162_amd import inputs as I  # noqa: E402


def _same(got, ref):
    assert (got.status, got.sizes, got.states_expanded, got.candidates) == (
        ref.status, ref.sizes, ref.states_expanded, ref.candidates)
    if ref.layers is not None:
        assert len(got.layers) == len(ref.layers)
        for a, b in zip(got.layers, ref.layers):
            assert np.array_equal(a, b)


@pytest.mark.parametrize("n,m", [(2, 1), (3, 2), (4, 1), (5, 2), (6, 1), (7, 2), (8, 3), (9, 2), (10, 2)])
@pytest.mark.parametrize("directed", [False, True])
def test_random_sets(n, m, directed, oracle_c):
    r = I.rng_for(n, seed=77 + m)
    gens = I.random_perms_with_inverses(n, m, r)
    if directed:
        gens = gens[:m]
    start = [int(x) for x in r.permutation(n)]
    kw = dict(max_layers=512, start=start, export_layers=60_000, allow_directed=directed)
    got = api.growth_ex(n, gens, **kw)
    _same(got, api.growth_ex(n, gens, packed_sort=True, **kw))
    if n <= 9:
        exp, rc, _ = oracle_c.growth(n, gens, max_layers=512)
        assert got.sizes == exp and got.status == rc


# large steps and steps from the unseen side: many generators (k = 45, 55),
# few (LRX: long runs of middling layers), a directed set
@pytest.mark.parametrize("n,fam", [(10, "all_transpositions"), (11, "all_transpositions"), (11, "pancake"), (10, "lrx"),
                                   (11, "lx"), (10, "coxeter")])
def test_large_steps(n, fam):
    gens = I.family(fam, n)
    kw = dict(max_layers=512, export_layers=20_000, allow_directed=fam == "lx")
    _same(api.growth_ex(n, gens, **kw), api.growth_ex(n, gens, packed_sort=True, **kw))
    kept = api.growth_ex(n, gens, keep_all_layers=True, max_layers=512, allow_directed=fam == "lx")
    assert sum(kept.sizes) == np.prod(np.arange(1, n + 1))


@pytest.mark.parametrize("frontier", [1, 4_000, 9_300, 200_000, 1_500_000])
@pytest.mark.parametrize("directed", [False, True])
def test_stop_rules_in_chains_and_large_steps(frontier, directed):
    n = 11
    gens = I.random_perms_with_inverses(n, 2, I.rng_for(5, seed=9))[: 2 if directed else 4]
    for rule in (dict(max_frontier=frontier), dict(max_layers=frontier % 17 + 2)):
        kw = dict(dict(max_layers=512), allow_directed=directed, **rule) if "max_layers" not in rule else dict(
            allow_directed=directed, **rule)
        _same(api.growth_ex(n, gens, **kw), api.growth_ex(n, gens, packed_sort=True, **kw))


def test_subgroups_and_reused_engine():
    """Orbits smaller than n! (the unseen states are never reached), and
    bitmaps left over from other jobs on the same engine."""
    eng = api.Engine()
    even = I.family("three_cycles", 9)                                   # A_9
    blocks = [list(range(1, 5)) + [0] + list(range(5, 11)), [4, 0, 1, 2, 3] + list(range(5, 11)),
              list(range(5)) + list(range(6, 11)) + [5], list(range(5)) + [10] + list(range(5, 10))]  # Z_5 x Z_6
    for n, gens in [(10, I.pancake(10)), (9, even), (11, blocks), (10, I.pancake(10)), (9, even)]:
        _same(eng.run(n, gens, max_layers=512), api.growth_ex(n, gens, max_layers=512, packed_sort=True))
    eng.close()

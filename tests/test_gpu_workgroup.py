"""The one-workgroup engine (CG_SMALL_JOB, batches) against the CPU oracle:
states of up to eight entries by table lookups, n = 9 in LDS, n = 10 in
memory; steps from the side of the unseen states (many generators); directed
sets, starts and stop rules. Tolerance: none (exact integers)."""

import pytest

pytestmark = pytest.mark.gpu

from paper_2509_19162_amd import api  # noqa: E402
from paper_2509_19162_amd import inputs as I  # noqa: E402


@pytest.mark.parametrize("n", [1, 2, 3, 5, 7, 8, 9, 10])
@pytest.mark.parametrize("m,directed", [(1, False), (2, True), (3, False)])
def test_random_sets_starts_and_rules(n, m, directed, oracle_c):
    r = I.rng_for(n, seed=31 + m)
    gens = I.random_perms_with_inverses(n, m, r)
    gens = gens[:m] if directed else gens
    start = [int(x) for x in r.permutation(n)]
    eng = api.Engine()
    for kw in (dict(max_layers=512), dict(max_layers=6), dict(max_layers=512, max_frontier=200)):
        got = eng.run(n, gens, start=start, allow_directed=directed, small_job=True, **kw)
        ref = api.growth_ex(n, gens, start=start, allow_directed=directed, packed_sort=True, **kw)
        assert (got.status, got.sizes, got.states_expanded, got.candidates) == (
            ref.status, ref.sizes, ref.states_expanded, ref.candidates)
    if n <= 8:
        exp, rc, _ = oracle_c.growth(n, gens, max_layers=512)
        assert eng.run(n, gens, max_layers=512, allow_directed=directed, small_job=True).sizes == exp
    eng.close()


@pytest.mark.parametrize("fam", ["all_transpositions", "reversals", "pancake", "coxeter", "three_cycles"])
@pytest.mark.parametrize("n", [8, 9])
def test_families(n, fam, oracle_c):
    gens = I.family(fam, n)
    exp, rc, _ = oracle_c.growth(n, gens, max_layers=512)
    r = api.growth_ex(n, gens, max_layers=512, small_job=len(gens) <= 128)
    assert r.sizes == exp and r.status == rc


def test_batches_mix_the_ranges(oracle_c):
    """Jobs of n = 10, 9 and up to 8 in one batch, and each range missing:
    the launch graph has one kernel or two."""
    pool = {n: [(n, I.family(f, n)) for f in ("pancake", "star", "lrx")] for n in (6, 8, 9, 10)}
    for ns in [(6, 8, 9, 10), (9,), (10,), (8, 10), (6, 9)]:
        jobs = [j for n in ns for j in pool[n]] * 2
        for got in (api.growth_batch(jobs, max_layers=512), api.growth_batch_noalloc(jobs, max_layers=512)):
            for (n, g), r in zip(jobs, got):
                assert r.sizes == oracle_c.growth(n, g, max_layers=512)[0]


@pytest.mark.parametrize("fam", ["coxeter", "all_transpositions", "reversals"])
def test_ten_entries_many_rounds(fam):
    """n = 10 with crowded neighbours (adjacent swaps: most lie in one part of
    the bitmap) and with many generators (lists fill up within a state)."""
    gens = I.family(fam, 10)
    ref = api.growth_ex(10, gens, max_layers=512, packed_sort=True)
    for r in (api.growth_ex(10, gens, max_layers=512, small_job=True),
              api.growth_batch_noalloc([(10, gens)], max_layers=512)[0]):
        assert r.sizes == ref.sizes and r.status == ref.status

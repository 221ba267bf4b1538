"""One-workgroup growths on S_1 to S_8, whose bitmaps have n! bits (a last
word with bits of no state among them), against the oracle. Tolerance: none
(exact integers)."""

import pytest

pytestmark = pytest.mark.gpu

from paper_2509_19162_amd import api  # noqa: E402
from paper_2509_19162_amd import inputs as I  # noqa: E402


def _sets(n):
    rng = I.rng_for(n, seed=61)
    yield [list(range(n))]
    if n > 1:
        yield [I.left_shift(n)]
        for f in ("coxeter", "pancake", "star", "all_transpositions"):
            yield I.family(f, n)
        for m in (1, 2, 4):
            yield I.random_perms_with_inverses(n, m, rng)
            yield [[int(x) for x in rng.permutation(n)] for _ in range(m)]
    if n > 2:
        yield I.lrx(n)
        yield I.lx(n)
        yield I.random_involutions(n, 3, rng)


@pytest.mark.parametrize("n", range(1, 9))
def test_growths(n, oracle_c):
    jobs = []
    for gens in _sets(n):
        for rule in ({}, {"max_layers": 3}, {"max_frontier": 2}, {"max_frontier": 40}):
            kw = dict({"max_layers": 256}, **rule)
            exp, rc, _ = oracle_c.growth(n, gens, max_layers=kw["max_layers"], max_frontier=kw.get("max_frontier", 0))
            start = [int(x) for x in I.rng_for(len(jobs), seed=62).permutation(n)]
            r = api.growth_ex(n, gens, small_job=True, allow_directed=True, start=start, **kw)
            assert (r.sizes, r.status) == (exp, rc), (gens, rule)
            jobs.append(((n, gens, kw.get("max_frontier"), kw["max_layers"]), (exp, rc)))
    for f in (api.growth_batch, api.growth_batch_noalloc):
        got = f([j for j, _ in jobs], allow_directed=True)
        assert [(r.sizes, r.status) for r in got] == [e for _, e in jobs]


def test_a_group_of_120_states_does_not_go_over_40320_bits():
    """S_5 under L, R, X: 11 layers, 130 us over the bits of S_8, 35 over 120."""
    eng = api.Engine()
    small = min(eng.run(5, I.lrx(5), small_job=True).device_ms for _ in range(20))
    large = min(eng.run(8, I.lrx(8), max_layers=11, small_job=True).device_ms for _ in range(20))
    assert small < 0.75 * large
    eng.close()

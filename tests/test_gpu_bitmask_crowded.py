"""Bitmask growths whose layers crowd in part of the ranks: they are tested
directly, layers spread evenly go through lists (some of which overrun), and
sizes are those of the rank bitmap or the sort. Tolerance: none (exact
integers)."""

import time

import pytest

pytestmark = pytest.mark.gpu

from paper_2509_19162_amd import api  # noqa: E402
from paper_2509_19162_amd import inputs as I  # noqa: E402

SETS = [(11, f) for f in ("coxeter", "cyclic_coxeter", "star", "pancake", "lrx", "reversals", "all_transpositions")]
SETS += [(12, "lrx"), (12, "pancake"), (12, "star")]


@pytest.mark.parametrize("n,fam", SETS)
def test_whole_growths(n, fam):
    gens, start = I.family(fam, n), [int(x) for x in I.rng_for(n, seed=41).permutation(n)]
    got = api.growth_ex(n, gens, max_layers=256, start=start, bitmask=True)
    ref = api.growth_ex(n, gens, max_layers=256, start=start)
    assert (got.status, got.sizes, got.states_expanded, got.candidates) == (
        ref.status, ref.sizes, ref.states_expanded, ref.candidates)


@pytest.mark.parametrize("n,fam,ms", [(13, "coxeter", 18), (11, "reversals", 18), (12, "reversals", 28)])
def test_crowded_layers_are_not_made_twice(n, fam, ms):
    """Up to a layer of 3e6 states: direct tests take 9, 12 and 17 ms; lists
    that overran took 32, 26 and 43."""
    eng = api.Engine()
    runs = [eng.run(n, I.family(fam, n), max_layers=256, max_frontier=3_000_000, bitmask=True) for _ in range(4)]
    assert min(r.device_ms for r in runs) < ms
    eng.close()


def test_short_growths_do_not_look_for_scattering_generators():
    """78 generators looked at on the host took 1.3 ms of a call of 2.1."""
    eng, gens = api.Engine(), I.all_transpositions(13)

    def best(g):
        times = []
        for _ in range(10):
            t = time.perf_counter()
            eng.run(13, g, max_layers=4, bitmask=True)
            times.append(time.perf_counter() - t)
        return min(times)

    assert best(gens) - best(gens[:1]) < 2.1e-3
    eng.close()

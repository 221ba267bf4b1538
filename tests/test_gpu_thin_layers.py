"""One-workgroup growths of S_10 whose layers are thin (a list of states) and
those that pass from thin layers to whole bitmaps, against the rank bitmap.
Tolerance: none (exact integers)."""

import pytest

pytestmark = pytest.mark.gpu

from paper_2509_19162_amd import api  # noqa: E402
from paper_2509_19162_amd import inputs as I  # noqa: E402

CYCLES = I.parse_cycles(10, "(0,1,2,3,4)(5,6,7)(8,9)")  # order 30


def _sets():
    rng = I.rng_for(5, seed=31)
    yield "one of order 30", [CYCLES], True
    yield "one involution", [I.transposition(10, 2, 7)], False
    yield "no generator", [list(range(10))], False
    yield "ring", [I.left_shift(10), I.inverse(I.left_shift(10))], False
    # commuting transpositions: an orbit of 32
    yield "cube", [I.transposition(10, i, i + 1) for i in range(0, 10, 2)], False
    # S_8 on the first entries: thin, then not, then thin
    yield "S_8", [g + [8, 9] for g in I.coxeter(8)], False
    yield "S_10 lx", I.lx(10), True
    yield "S_10 pancake", I.pancake(10), False
    yield "S_10 transpositions", I.all_transpositions(10), False
    yield "S_10 random", I.random_perms_with_inverses(10, 60, rng), False


@pytest.mark.parametrize("name,gens,directed", list(_sets()), ids=lambda x: x if isinstance(x, str) else "")
def test_growths(name, gens, directed):
    start = [int(x) for x in I.rng_for(7, seed=31).permutation(10)]
    for rule in ({}, {"max_layers": 3}, {"max_layers": 9}, {"max_frontier": 1}, {"max_frontier": 150},
                 {"max_frontier": 4_000}):
        kw = dict({"max_layers": 256, "start": start, "allow_directed": directed}, **rule)
        got, ref = api.growth_ex(10, gens, small_job=True, **kw), api.growth_ex(10, gens, packed_sort=True, **kw)
        assert (got.status, got.sizes, got.states_expanded, got.candidates) == (
            ref.status, ref.sizes, ref.states_expanded, ref.candidates), rule


def test_a_thin_layer_does_not_go_over_the_bitmaps():
    """30 layers of one state: over the bitmaps each took 285 us."""
    eng = api.Engine()
    ms = min(eng.run(10, [CYCLES], small_job=True, allow_directed=True).device_ms for _ in range(5))
    assert len(eng.run(10, [CYCLES], small_job=True, allow_directed=True).sizes) == 30
    assert ms < 30 * 0.025
    eng.close()

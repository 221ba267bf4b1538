"""The hash-bucket engine proper (permutations of 13 to 16 entries, repeated
entries, binary states): stop rules at its limits, export cuts, one engine for
many jobs, and the ways back from plans that expected too little. The same
for the rank bitmap and the bitmask engine's lists. Against the sort path,
state by state. Tolerance: none (exact integers)."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from paper_2509_19162_amd import api  # noqa: E402
from paper_2509_19162_amd import inputs as I  # noqa: E402

MULTI14 = [4, 4, 3, 3, 3, 2, 2, 2, 1, 1, 1, 0, 0, 0]
JOBS = [(13, "lrx", None), (16, "star", None), (16, "lrx", None), (14, "coxeter", MULTI14),
        (24, "lrx", [0] * 12 + [1] * 12), (26, "reversals", [0] * 20 + [1] * 6)]


def _same(got, ref):
    assert (got.status, got.sizes, got.states_expanded, got.candidates) == (
        ref.status, ref.sizes, ref.states_expanded, ref.candidates)
    if ref.layers is not None:
        assert len(got.layers) == len(ref.layers)
        for a, b in zip(got.layers, ref.layers):
            assert np.array_equal(a, b)


@pytest.mark.parametrize("limit", [1, 3, 500, 4_608, 9_215, 9_216, 9_217, 16_384, 16_385, 400_000])
@pytest.mark.parametrize("n,fam,start", JOBS)
def test_stop_rules(n, fam, start, limit):
    """Inside and between the one-workgroup layers (9216 states of three
    layers, 16384 candidates) and the partitioned ones."""
    gens = I.family(fam, n)
    kw = dict(start=start, max_layers=256, max_frontier=limit, export_layers=50_000)
    got = api.growth_ex(n, gens, **kw)
    _same(got, api.growth_ex(n, gens, packed_sort=True, **kw))
    kw = dict(start=start, max_layers=limit % 20 + 1, max_frontier=1_000_000)
    _same(api.growth_ex(n, gens, **kw), api.growth_ex(n, gens, packed_sort=True, **kw))


@pytest.mark.parametrize("cap", [0, 1, 2, 9_000, 40_000, 300_000])
@pytest.mark.parametrize("n,fam,start", JOBS)
def test_export_capacity_cuts_layers(n, fam, start, cap):
    kw = dict(start=start, max_layers=256, max_frontier=200_000, export_layers=cap)
    _same(api.growth_ex(n, I.family(fam, n), **kw), api.growth_ex(n, I.family(fam, n), packed_sort=True, **kw))


def test_one_engine_for_many_jobs():
    """Buffers, bucket tables, tags and counters left by one job do not reach
    the next."""
    eng = api.Engine()
    for frontier in (100_000, 1_500_000, 3_000):
        for n, fam, start in JOBS:
            gens = I.family(fam, n)
            kw = dict(start=start, max_layers=512, max_frontier=frontier)
            ref = api.growth_ex(n, gens, packed_sort=True, **kw)
            _same(eng.run(n, gens, **kw), ref)
            _same(eng.run(n, gens, keep_all_layers=True, **kw), ref)
    eng.close()


@pytest.mark.parametrize("options", [{}, {"export_layers": 300_000}, {"keep_all_layers": True}])
@pytest.mark.parametrize("factor", [0.5, 0.1, 0.001])
@pytest.mark.parametrize("n,fam,start", JOBS)
def test_layers_larger_than_expected(n, fam, start, factor, options, monkeypatch):
    """The buckets once more into a larger buffer; tables that overrun: the
    layer again with more buckets."""
    gens = I.family(fam, n)
    kw = dict(start=start, max_layers=512, max_frontier=1_000_000, **options)
    ref = api.growth_ex(n, gens, packed_sort=True, **kw)
    monkeypatch.setenv("CG_EXPECT_FACTOR", str(factor))
    _same(api.growth_ex(n, gens, **kw), ref)


@pytest.mark.parametrize("options", [{}, {"export_layers": 300_000}, {"keep_all_layers": True}])
@pytest.mark.parametrize("factor", [0.7, 0.2, 0.0])
@pytest.mark.parametrize("n,fam,start", JOBS + [(10, "pancake", None), (11, "lrx", None), (12, "star", None)])
def test_parts_that_overrun(n, fam, start, factor, options, monkeypatch):
    """Hash buckets: the sort path goes on. Rank bitmap: the bitmap is built
    again and layers take small steps."""
    gens = I.family(fam, n)
    kw = dict(start=start, max_layers=512, max_frontier=1_000_000, **options)
    ref = api.growth_ex(n, gens, packed_sort=True, **kw)
    monkeypatch.setenv("CG_PART_FACTOR", str(factor))
    _same(api.growth_ex(n, gens, **kw), ref)


@pytest.mark.parametrize("factor", [0.7, 0.2, 0.0])
@pytest.mark.parametrize("n,gens", [(11, I.random_perms_with_inverses(11, 2, I.rng_for(1, seed=51))),
                                    (11, I.pancake(11)), (12, I.random_perms_with_inverses(12, 2, I.rng_for(2, seed=51)))],
                         ids=["S_11 random", "S_11 pancake", "S_12 random"])
def test_lists_that_overrun(n, gens, factor, monkeypatch):
    """Bitmask engine: the piece is tested directly."""
    ref = api.growth_ex(n, gens, max_layers=256)
    monkeypatch.setenv("CG_PART_FACTOR", str(factor))
    _same(api.growth_ex(n, gens, max_layers=256, bitmask=True), ref)


@pytest.mark.parametrize("n,fam,directed", [(7, "coxeter", False), (9, "pancake", False), (10, "coxeter", False),
                                            (10, "lx", True), (11, "lrx", False), (12, "star", False), (13, "lrx", False),
                                            (16, "star", False)])
def test_rank_sorts_of_the_sort_path(n, fam, directed, monkeypatch):
    """Chunks of any size turn the other engines off: 32-bit ranks (full and
    incremental) up to n = 12, 64-bit ranks beyond."""
    gens = I.lx(n) if fam == "lx" else I.family(fam, n)
    kw = dict(max_layers=512, max_frontier=300_000, allow_directed=directed, export_layers=50_000)
    ref = api.growth_ex(n, gens, packed_sort=True, **kw)
    _same(api.growth_ex(n, gens, **kw), ref)
    monkeypatch.setenv("CG_CHUNK_CANDIDATES", str(10 ** 17))
    got = api.growth_ex(n, gens, profile=True, **kw)
    _same(got, ref)
    assert "dedup_compact" in got.kstats and "bucket_dedup" not in got.kstats
    monkeypatch.setenv("CG_RANK_FULL", "1")
    _same(api.growth_ex(n, gens, **kw), ref)

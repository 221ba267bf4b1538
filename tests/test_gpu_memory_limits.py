"""Growths under a limit on device memory (CG_DEVICE_BYTES): wherever the
sort path finishes, the default engines do as well, with its results, and the
states of the layers are the same. Tolerance: none (exact integers)."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from paper_2509_19162_amd import _native as N  # noqa: E402
from paper_2509_19162_amd import api  # noqa: E402
from paper_2509_19162_amd import inputs as I  # noqa: E402

LIMITS_MIB = (2, 4, 8, 12, 16, 24, 32, 48, 64, 96, 128, 192, 256, 384, 512, 1024)
OPTIONS = [{}, {"export_layers": 2_000_000}, {"keep_all_layers": True},
           {"keep_all_layers": True, "export_layers": 2_000_000}]


def _run(monkeypatch, sort_path, n, gens, **kw):
    """The growth, or None when device memory is too short for it. Chunks of
    any size turn the other engines off."""
    with monkeypatch.context() as m:
        if sort_path:
            m.setenv("CG_CHUNK_CANDIDATES", str(10 ** 17))
        try:
            return api.growth_ex(n, gens, max_layers=512, **kw)
        except api.CGError as e:
            assert e.code == N.CG_E_NOMEM
            return None


def _same(got, ref):
    assert (got.status, got.sizes, got.states_expanded, got.candidates) == (
        ref.status, ref.sizes, ref.states_expanded, ref.candidates)
    for a, b in zip(got.layers or [], ref.layers or []):
        assert np.array_equal(a, b)


def _finishes_where_sorting_does(monkeypatch, n, gens, **kw):
    ref = _run(monkeypatch, True, n, gens, **kw)
    finished = 0
    for mib in LIMITS_MIB:
        monkeypatch.setenv("CG_DEVICE_BYTES", str(api.memory_stats()["held_bytes"] + (mib << 20)))
        by_sort = _run(monkeypatch, True, n, gens, **kw)
        got = _run(monkeypatch, False, n, gens, **kw)
        assert got is not None or by_sort is None, mib
        if got is not None:
            _same(got, ref)
            finished += 1
    assert finished


@pytest.mark.parametrize("options", OPTIONS)
@pytest.mark.parametrize("n,fam,frontier", [(10, "pancake", None), (11, "lrx", 300_000), (12, "pancake", 3_000_000)])
def test_permutations_over_the_rank_bitmap(n, fam, frontier, options, monkeypatch):
    _finishes_where_sorting_does(monkeypatch, n, I.family(fam, n), max_frontier=frontier, **options)


@pytest.mark.parametrize("options", OPTIONS)
def test_directed_permutations(options, monkeypatch):
    _finishes_where_sorting_does(monkeypatch, 10, I.lx(10), allow_directed=True, **options)


@pytest.mark.parametrize("options", OPTIONS)
@pytest.mark.parametrize("n,fam,start,frontier", [
    (13, "lrx", None, 1_000_000), (16, "star", None, 1_000_000), (24, "lrx", [0] * 12 + [1] * 12, None),
    (14, "coxeter", [4, 4, 3, 3, 3, 2, 2, 2, 1, 1, 1, 0, 0, 0], 1_000_000)])
def test_layers_by_hash_buckets(n, fam, start, frontier, options, monkeypatch):
    _finishes_where_sorting_does(monkeypatch, n, I.family(fam, n), start=start, max_frontier=frontier, **options)


def test_hand_over_holds_one_copy_of_a_layer(monkeypatch):
    """C(24, 12) = 2,704,156 binary states in some 200 layers: two of these,
    one copy and the sort path's chunks fit 5 MiB."""
    gens, start = I.lrx(24), [0] * 12 + [1] * 12
    ref = api.growth_ex(24, gens, max_layers=512, start=start)
    monkeypatch.setenv("CG_DEVICE_BYTES", str(api.memory_stats()["held_bytes"] + (5 << 20)))
    _same(api.growth_ex(24, gens, max_layers=512, start=start), ref)


def test_last_small_layers_without_room_for_a_run(monkeypatch):
    """All 2,704,156 states kept in 52 MiB: the last layers are small, but
    not even 9216 more states fit; they are not paid for with a second
    growth by sorting (its 209 layers)."""
    gens, start = I.lrx(24), [0] * 12 + [1] * 12
    kw = dict(max_layers=512, start=start, keep_all_layers=True, profile=True)
    ref = api.growth_ex(24, gens, **kw)
    monkeypatch.setenv("CG_DEVICE_BYTES", str(api.memory_stats()["held_bytes"] + (52 << 20)))
    got = api.growth_ex(24, gens, **kw)
    _same(got, ref)
    assert got.kstats.get("dedup_compact", {"launches": 0})["launches"] < 100


@pytest.mark.parametrize("mib", [4, 24, 140, 300])
def test_batches_of_n_10_with_few_slots(mib, monkeypatch):
    """100 jobs (one workgroup each) whose bitmaps alone take 130 MiB: with
    less, they take turns."""
    jobs = [(10, I.random_perms_with_inverses(10, 2, I.rng_for(i, seed=22))) for i in range(100)]
    ref = api.growth_batch_noalloc(jobs)
    api.release_cached_memory()
    monkeypatch.setenv("CG_DEVICE_BYTES", str(api.memory_stats()["held_bytes"] + (mib << 20)))
    for _ in range(2):
        got = api.growth_batch(jobs)
        assert [(r.status, r.sizes, r.states_expanded) for r in got] == [(r.status, r.sizes, r.states_expanded) for r in ref]
    monkeypatch.delenv("CG_DEVICE_BYTES")
    assert [r.sizes for r in api.growth_batch(jobs)] == [r.sizes for r in ref]


@pytest.mark.parametrize("mib", [24, 64, 200])
def test_bitmask_engine_without_room_for_lists(mib, monkeypatch):
    """Three bitmaps of 5 MB, lists of some 90 MB where they fit."""
    gens = I.random_perms_with_inverses(11, 2, I.rng_for(1, seed=51))
    ref = api.growth_ex(11, gens, max_layers=256)
    monkeypatch.setenv("CG_DEVICE_BYTES", str(api.memory_stats()["held_bytes"] + (mib << 20)))
    _same(api.growth_ex(11, gens, max_layers=256, bitmask=True), ref)

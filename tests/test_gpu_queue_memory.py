"""The queue's accounts of device memory: what a job held at most is what the
queue reports, and stays within what it charged."""

import pytest

pytestmark = pytest.mark.gpu

from paper_2509_19162_amd import api  # noqa: E402
from paper_2509_19162_amd import inputs as I  # noqa: E402

FIXED = 16 << 20  # the lanes' fixed buffers


@pytest.mark.parametrize("n,fam,frontier,candidates", [
    (15, "lrx", 2_000_000, 100_000),  # handed to the sort path, which frees the buckets' buffers
    (13, "lrx", 1_000_000, None),     # the bitmask engine
    (11, "pancake", None, None)])     # the rank bitmap
def test_peak_held_is_what_was_held(n, fam, frontier, candidates, monkeypatch):
    if candidates:
        monkeypatch.setenv("CG_HASH_CANDIDATES", str(candidates))
    gens = I.family(fam, n)
    with api.GrowthQueue() as q:
        base = api.memory_stats(reset_peak=True)["held_bytes"]
        q.wait(q.submit(n, gens, max_layers=256, max_frontier=frontier), timeout_s=120)
        held = api.memory_stats()["peak_held_bytes"] - base
        st = q.stats()
    assert held > FIXED
    # (the lanes make their fixed buffers before or after `base` is read)
    assert abs(st["peak_held_bytes"] - held) <= FIXED
    assert st["over_bound"] == 0


@pytest.mark.parametrize("n,fam,kw", [
    (11, "lrx", {"max_frontier": 100_000}), (11, "lrx", {"max_frontier": 20_000}), (11, "star", {"max_frontier": 5_000}),
    (11, "coxeter", {"max_layers": 20}), (11, "pancake", {}), (10, "star", {"max_frontier": 1_000}), (10, "reversals", {}),
    (11, "lx", {"allow_directed": True, "max_frontier": 50_000})])
def test_rank_bitmap_jobs_stay_within_their_charge(n, fam, kw):
    gens = I.lx(n) if fam == "lx" else I.family(fam, n)
    kw = dict({"max_layers": 256}, **kw)
    with api.GrowthQueue() as q:
        r = q.wait(q.submit(n, gens, **kw), timeout_s=120)
        st = q.stats()
    assert st["over_bound"] == 0
    assert st["peak_held_bytes"] <= st["peak_charged_bytes"] + FIXED
    ref = api.growth_ex(n, gens, packed_sort=True, **kw)
    assert (r.sizes, r.status) == (ref.sizes, ref.status)

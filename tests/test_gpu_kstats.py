"""Kernel times of a growth that is handed to the sort path: nine or more
kinds of kernels for eight places. None of their time is lost."""

import pytest

pytestmark = pytest.mark.gpu

from paper_2509_19162_amd import api  # noqa: E402
from paper_2509_19162_amd import inputs as I  # noqa: E402


@pytest.mark.parametrize("n,fam,start,frontier,longest", [
    (13, "lrx", None, 6_000_000, {"small_layers", "bucket_dedup", "sort_pass", "dedup_compact"}),
    (14, "coxeter", [4, 4, 3, 3, 3, 2, 2, 2, 1, 1, 1, 0, 0, 0], 1_500_000,
     {"bucket_dedup", "sort_pass", "sort_pass_expand", "dedup_compact"})])
def test_kinds_beyond_the_places(n, fam, start, frontier, longest, monkeypatch):
    monkeypatch.setenv("CG_HASH_CANDIDATES", "8000000")
    r = api.growth_ex(n, I.family(fam, n), max_layers=512, start=start, max_frontier=frontier, profile=True)
    assert len(r.kstats) <= 8 and longest <= set(r.kstats)
    # kinds of least time are part of "aux": more launches than layers in all
    assert sum(k["launches"] for k in r.kstats.values()) > 2 * len(r.sizes)

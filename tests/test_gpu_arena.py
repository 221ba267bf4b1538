"""The regions that device buffers are carved from: growths of ordinary size
do not make the library reserve most of the device's memory (which takes
seconds), large ones do, and all of it is given back."""

import gc

import pytest

pytestmark = pytest.mark.gpu

from paper_2509_19162_amd import api  # noqa: E402
from paper_2509_19162_amd import inputs as I  # noqa: E402


def _arena():
    return api.memory_stats()["arena_bytes"]


def test_ordinary_growths_reserve_a_small_region():
    gc.collect()
    api.release_cached_memory()
    if _arena():
        pytest.skip("buffers of another test are alive")
    cycle = [[(i + 1) % 11 for i in range(11)]]
    assert api.growth_ex(11, cycle, allow_directed=True).sizes == [1] * 11
    assert _arena() == 0
    eng = api.Engine()
    kw = dict(max_layers=64, max_frontier=3_000_000)
    got = eng.run(16, I.lrx(16), **kw)
    assert 0 < _arena() <= 16 << 30
    # beyond it: the large region, beside buffers that live in the first
    assert api.growth_ex(14, I.lrx(14), max_layers=3, bitmask=True).sizes == [1, 3, 6]
    assert _arena() > 64 << 30
    again = eng.run(16, I.lrx(16), **kw)
    ref = api.growth_ex(16, I.lrx(16), packed_sort=True, **kw)
    assert got.sizes == again.sizes == ref.sizes
    eng.close()
    api.release_cached_memory()
    assert _arena() == 0

"""Streams and pinned memory kept between calls: growths from several threads
(own streams and the caller's), one-workgroup jobs, batches and the release of
everything cached, all at once, against the CPU oracle. Exact integers."""

import threading

import pytest

pytestmark = pytest.mark.gpu

from paper_2509_19162_amd import api  # noqa: E402
from paper_2509_19162_amd import inputs as I  # noqa: E402


@pytest.mark.parametrize("threads", [2, 8])
def test_threads_and_release(threads, oracle_c):
    import torch

    cases = [(n, I.family(f, n)) for n in (5, 7, 8) for f in ("coxeter", "pancake", "star")]
    exp = [oracle_c.growth(n, g, max_layers=512)[0] for n, g in cases]
    bad = []

    def work(t):
        stream = torch.cuda.Stream() if t % 2 else None
        for rep in range(6):
            for (n, g), e in zip(cases, exp):
                for kw in ({}, {"small_job": True}, {"packed_sort": True}, {"bitmask": True}):
                    if api.growth_ex(n, g, max_layers=512, stream=stream, **kw).sizes != e:
                        bad.append((t, n, kw))
            if t == 0:
                api.release_cached_memory()
            if t == 1:
                got = api.growth_batch(cases, max_layers=512)
                if [r.sizes for r in got] != exp:
                    bad.append((t, "batch"))

    ts = [threading.Thread(target=work, args=(t,)) for t in range(threads)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not bad

"""The device slots of n = 10 jobs without allocation: as many as the array
holds are in use at once, and every number of jobs gives the same growths."""

import time

import pytest

pytestmark = pytest.mark.gpu

from paper_2509_19162_amd import api  # noqa: E402
from paper_2509_19162_amd import inputs as I  # noqa: E402


def _jobs(count):
    return [(10, I.random_perms_with_inverses(10, 2, I.rng_for(i, seed=21))) for i in range(count)]


@pytest.mark.parametrize("count", [1, 2, 44, 45, 46, 47, 91])
def test_growths_for_every_number_of_slots(count):
    jobs = _jobs(count)
    got, ref = api.growth_batch_noalloc(jobs), api.growth_batch(jobs)
    assert [(r.status, r.sizes, r.states_expanded) for r in got] == [(r.status, r.sizes, r.states_expanded) for r in ref]


def test_growths_beside_the_most_layer_sizes():
    """2^21 recorded layer sizes leave the slots the least room."""
    jobs = _jobs(40) + [(7, I.coxeter(7))] * 4056
    got = api.growth_batch_noalloc(jobs, max_layers=512)
    ref = api.growth_batch(jobs, max_layers=512)
    assert [(r.status, r.sizes) for r in got] == [(r.status, r.sizes) for r in ref]


def test_35_jobs_run_side_by_side():
    """In two rounds they would take twice as long as 28."""
    def best(jobs):
        times = []
        for _ in range(5):
            t = time.perf_counter()
            api.growth_batch_noalloc(jobs)
            times.append(time.perf_counter() - t)
        return min(times)

    assert best(_jobs(35)) < 1.3 * best(_jobs(28))

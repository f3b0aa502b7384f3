"""A tick that outlasts its jobs: queued jobs take the places of finished ones
several times within it, in slots and arena space that were theirs, with more
image bytes than the pinned memory holds at once.  Every result equals the
oracle's, whatever the tick."""
import numpy as np
import pytest

from tests.test_gpu_server import KEYS, oracle_moments, run, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def jobs_and_oracle():
    g = np.random.default_rng(3)
    sizes = [1, 7, 511, 512, 4097, 20001, 70003]
    jobs = [(i, int(sizes[i % 7] if i % 3 else g.integers(1, 3000)), int(g.integers(0, 40)) if i % 5 else 0,
             float(5 + 1.5 * i), 0.1 * (i % 3 - 1)) for i in range(60)]
    return jobs, [oracle_moments(j) for j in jobs]


@pytest.mark.parametrize("tick", [1, 9, 4000])
def test_places_taken_within_a_tick(jobs_and_oracle, tick):
    jobs, want = jobs_and_oracle
    say("tick", tick)
    got = run(jobs, arena_bytes=3 * 2 * 70016 + 3 * 2 * 25000, max_slots=5, k=tick)
    assert sorted(got) == [j[0] for j in jobs]
    for job, w in zip(jobs, want):
        for k in KEYS:
            assert got[job[0]][k] == w[k], (job, k)

"""Schedules of fewer than 1024 threads with images as large as their own
queues leave room for, dense so that the images fill it: accepted, and every
count equals the oracle's.  Schedules of 1024 threads with images of any size:
several steps per launch, as with the largest, blocked or not."""
import pytest

from paper_1706_01094_amd.mclg import Lattice
from tests.test_gpu_register_steps import run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("threads", [64, 256, 768, 960, 1024])
@pytest.mark.parametrize("L", [3001, 100003])
def test_largest_images(threads, L):
    run(L, (3, 20), rho=95.0, u0=0.25, schedule=(1, threads, 160 << 10))


@pytest.mark.parametrize("lds", [0, 16 << 10, 64 << 10, 96 << 10, 112 << 10])
@pytest.mark.parametrize("L", [3001, 100003])
def test_small_images(lds, L):
    run(L, (3, 20), rho=40.0, schedule=(1, 1024, lds))


@pytest.mark.parametrize("lds", [0, 96 << 10, 128 << 10])
def test_blocked_with_small_images(lds):
    L = 1 << 20
    a, b = (Lattice(L, 3, rho=30.0, u0=0.05) for _ in range(2))
    a.set_schedule(1, 1024, lds)
    b.set_drain(1)
    assert b.step_plan(64) == {"launches": 64, "steps_per_launch": 1, "sites_per_lane": 0, "extra_sites": 0}
    a.set_blocked(64)
    p = a.step_plan(64)
    assert p["steps_per_launch"] > 1 and p["sites_per_lane"] > 0 and p["launches"] * p["steps_per_launch"] >= 64
    a.step(64)
    b.step(64)
    assert a.moments(digest=True) == b.moments(digest=True)
    a.close()
    b.close()

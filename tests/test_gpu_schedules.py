"""Schedules of fewer than 1024 threads with images as large as their own
queues leave room for, dense so that the images fill it: accepted, and every
count equals the oracle's."""
import pytest

from tests.test_gpu_register_steps import run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("threads", [64, 256, 768, 960, 1024])
@pytest.mark.parametrize("L", [3001, 100003])
def test_largest_images(threads, L):
    run(L, (3, 20), rho=95.0, u0=0.25, schedule=(1, threads, 160 << 10))

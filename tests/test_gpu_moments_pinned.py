"""mclg_moments of few and of many replicas (through pinned memory or the
workspace), with a segment per replica and with several, after steps that the
device's counters do not hold yet: the same sums as mclg_moments_noalloc's;
and a site that overflowed is reported either way."""
import numpy as np
import pytest
import torch

from paper_1706_01094_amd.mclg import E_RANGE, Lattice, MclgError

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,L", [(1, 5), (3, 40000), (4096, 9), (4097, 9)])
@pytest.mark.parametrize("digest", [False, True])
def test_same_as_the_device_results(n, L, digest):
    lat = Lattice(np.full(n, L, dtype=np.uint64), 3, rho=20.0, u0=0.1)
    lat.step(5)
    got = lat.moments(digest=digest)
    lat.step(3)
    got2 = lat.moments(digest=digest)
    out = torch.zeros(n * 33, dtype=torch.int64, device="cuda")
    lat.moments_to_device(out, digest=digest)
    assert lat.check() == 0
    torch.cuda.synchronize()
    rows = out.cpu().numpy().reshape(n, 33)
    assert all(m["t"] == 5 for m in got) and all(m["t"] == 8 for m in got2)
    assert [m["sum_N"] for m in got] == [m["sum_N"] for m in got2] == list(rows[:, 11])
    assert [m["max_N"] for m in got2] == list(rows[:, 15])
    assert [m["digest"] for m in got2] == list(rows.view(np.uint64)[:, 32])
    lat.close()


@pytest.mark.parametrize("n", [2, 4097])
def test_overflow_is_reported(n):
    counts = np.zeros((n, 3, 8), dtype=np.uint16)  # (replica by replica)
    counts[1, :, 3] = 30000
    lat = Lattice(np.full(n, 8, dtype=np.uint64), 3, counts=counts.reshape(-1))
    lat.step(1)
    with pytest.raises(MclgError) as e:
        lat.moments()
    assert e.value.code == E_RANGE
    lat.moments(allow_range=True)
    lat.close()

"""Calls recorded into a program's own HIP graph: every replay goes on from the
step that the one before it reached, and equals the same calls made one after
the other, also where the program read moments before it recorded them."""
import numpy as np
import pytest
import torch

from paper_1706_01094_amd.mclg import FLAG_GALILEAN, Lattice

pytestmark = pytest.mark.gpu

L5 = [700, 5, 4099, 60005, 256]


def two(L, blocked=0, **kw):
    pair = [Lattice(np.asarray(L, dtype=np.uint64), 9, rho=20.0, u0=0.1, **kw) for _ in range(2)]
    for l in pair:
        if blocked:
            l.set_blocked(blocked)
    return pair


def recorded(lat, calls):
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=lat.stream):
        calls()
    return g


def replay(g, lat):
    with torch.cuda.stream(lat.stream):
        g.replay()
    torch.cuda.synchronize()


def rows(lat, n=1):
    return torch.zeros(n * lat.n * 33, dtype=torch.int64, device="cuda")


@pytest.mark.parametrize("L", [[300], [60005], L5], ids=len)
@pytest.mark.parametrize("kw", [{}, dict(flags=FLAG_GALILEAN)], ids=str)
@pytest.mark.parametrize("warm", [0, 5])
def test_steps_and_moments(L, kw, warm):
    print("[gpu] case", L, kw, warm, flush=True)
    a, b = two(L, **kw)
    ra, rb = rows(a), rows(b)
    for l, r in ((a, ra), (b, rb)):
        l.moments_to_device(r, digest=True)
        if warm:
            l.step(warm)
        l.moments()

    def calls(l, r):
        l.step(7)
        l.moments_to_device(r, digest=True)

    g = recorded(a, lambda: calls(a, ra))
    for k in range(4):
        replay(g, a)
        calls(b, rb)
        assert b.check() == 0
        assert torch.equal(ra, rb), k
    a.close()
    b.close()


@pytest.mark.parametrize("L", [[300], [60005], L5[:3]], ids=len)
def test_logs(L):
    print("[gpu] case", L, flush=True)
    a, b = two(L)
    ra, rb = rows(a, 6), rows(b, 6)
    for l, r in ((a, ra), (b, rb)):
        l.step_log(2, 6, r, digest=True)
        l.moments()
    g = recorded(a, lambda: a.step_log(3, 6, ra, digest=True))
    for k in range(4):
        replay(g, a)
        b.step_log(3, 6, rb, digest=True)
        assert b.check() == 0
        assert torch.equal(ra, rb), k
    a.close()
    b.close()


@pytest.mark.parametrize("pending", [0, 5])
def test_blocked_replicas(pending):
    """The steps taken before need not be in the device's counters yet."""
    a, b = two(L5, blocked=8)
    ra, rb = rows(a), rows(b)
    for l, r in ((a, ra), (b, rb)):
        l.step(16)
        l.moments_to_device(r, digest=True)
        if pending:
            l.step(pending)
    torch.cuda.synchronize()
    g = recorded(a, lambda: a.step(16))
    for k in range(4):
        replay(g, a)
        b.step(16)
    a.moments_to_device(ra, digest=True)
    b.moments_to_device(rb, digest=True)
    assert a.check() == 0 and b.check() == 0
    torch.cuda.synchronize()
    assert torch.equal(ra, rb)
    a.close()
    b.close()

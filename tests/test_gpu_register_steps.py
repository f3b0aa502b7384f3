"""Several steps on sites held in registers (a lattice in one block's
registers, or tiles of one): every count equals the oracle's at the sizes
where the split can go wrong -- lattices of a lane, a wave and a block's
waves and one site more or less, lattices whose length is no multiple of 8
(streaming passes over the positions after the last site), lattices cut
between blocks, replicas that share an image or not, chunks with more
undecided sites than the queue holds, and every collision rule."""
import sys

import numpy as np
import pytest

import oracle as O
import synth
from paper_1706_01094_amd.mclg import E_RANGE, FLAG_GALILEAN, FLAG_NO_STREAM, Lattice

pytestmark = pytest.mark.gpu


def run(L, steps, rho=30.0, u0=0.1, counts=None, check=0, schedule=None, **kw):
    print("[gpu] case", L if np.ndim(L) == 0 else (len(L), L[:4]), steps, kw, flush=True)
    sys.stdout.flush()
    Ls = np.atleast_1d(np.asarray(L, dtype=np.uint64))
    rhos, u0s = np.broadcast_to(rho, Ls.shape), np.broadcast_to(u0, Ls.shape)
    init = {"counts": counts} if counts is not None else {"rho": rho, "u0": u0}
    g = Lattice(Ls, 83, **init, **kw)
    if schedule is not None:
        g.set_schedule(*schedule)
    o = O.OracleSim(Ls, 83, **kw)
    for r in range(len(Ls)):
        if counts is not None:
            o.init_counts(r, counts)
        else:
            o.init_poisson(r, float(rhos[r]), float(u0s[r]))
    for n in steps:
        g.step(n)
        o.step(n)
        assert g.check() == check
        for r in range(len(Ls)):
            a, b = g.counts(r, allow_range=check != 0), o.counts(r)
            bad = np.argwhere(a != b)
            assert not len(bad), (r, int(Ls[r]), n, len(bad), bad[:4].tolist())
    g.close()
    o.close()


@pytest.mark.parametrize("L", [1, 3, 8, 255, 256, 257, 1023, 1024, 1025, 4095, 4096, 4097, 8191, 16384])
def test_lattices_in_one_block(L):
    run(L, (1, 2, 30))


@pytest.mark.parametrize("L", [24569, 65536] + [70000 + k for k in range(1, 8)] + [300004, 1000003])
def test_lattices_between_blocks(L):
    run(L, (33, 5) if L > 200000 else (33, 120, 5))


@pytest.mark.parametrize("n,lo,hi", [(300, 250, 250), (600, 900, 900), (300, 1, 3000), (40, 513, 30000), (60, 400, 60000),
                                     (5, 600, 500000)])
def test_replicas(n, lo, hi):
    """Equal lattices (several per block, one image), uneven ones with images
    of their own, and short ones beside long ones cut between blocks."""
    rng = np.random.default_rng(n)
    L = rng.integers(lo, hi + 1, n)
    same = lo == hi
    rho = 30.0 if same else rng.uniform(5, 80, n)
    u0 = 0.1 if same else rng.uniform(-0.2, 0.2, n)
    run(L, (20, 3), rho=rho, u0=u0)


@pytest.mark.parametrize("L", [3001, 100003])
@pytest.mark.parametrize("kw", [dict(C=0), dict(C=1), dict(C=3, lam=(1, 2)), dict(C=20), dict(C=-1), dict(C=21), dict(n_max=24),
                                dict(flags=FLAG_NO_STREAM), dict(flags=FLAG_GALILEAN, lam=(3, 4)),
                                dict(flags=FLAG_GALILEAN, n_max=16), dict(C=30, flags=FLAG_GALILEAN)], ids=str)
def test_collision_rules(L, kw):
    run(L, (17, 4), u0=0.15, **kw)


@pytest.mark.parametrize("L", [2999, 60005])
def test_more_misses_than_the_queue_holds(L):
    """Every site far outside its image (built for the equilibrium of the
    same density): all draws come from the global rows."""
    counts = np.full((3, L), 60, dtype=np.uint16)
    run(L, (3, 20), counts=counts)


@pytest.mark.parametrize("L", [3001, 100003])
@pytest.mark.parametrize("lds", [(128 << 10) - 16, 128 << 10, 146176, 160 << 10])
def test_image_budgets_of_a_schedule(L, lds):
    """Around the smallest budget that takes these kernels, and the largest;
    dense, so that the images differ."""
    run(L, (3, 40), rho=90.0, u0=0.2, schedule=(1, 1024, lds))


@pytest.mark.parametrize("L", [900, 60005])
@pytest.mark.parametrize("kw", [dict(C=10), dict(C=3, lam=(2, 3)), dict(C=30), dict(C=10, lam=(3 << 20, 7 << 20))], ids=str)
def test_sites_without_a_row_among_others(L, kw):
    """Half of the sites past n_max, whose sub-collisions go one by one, none
    in the image; the last case rejects a third of the acceptance draws."""
    counts = np.full((3, L), 20, dtype=np.uint16)
    counts[1, ::3] = 19
    run(L, (1, 12), counts=counts, n_max=60, **kw)


@pytest.mark.parametrize("L", [500, 40003])
def test_overflow_is_flagged_and_kept(L):
    counts = synth.random_counts(L, seed=5)
    counts[:, L // 3] = 30000
    run(L, (12,), counts=counts, check=E_RANGE)


def test_no_flag_from_extra_sites():
    """The left half moves left, the right half right, 40000 particles a site:
    no site of the lattice ever holds more than 65535, but at the ends of a
    wave, whose values are wrong, the two meet.  No error is raised."""
    L, gap = 50000, 64
    counts = np.zeros((3, L), dtype=np.uint16)
    counts[0, gap:L // 2] = 40000
    counts[2, L // 2:L - gap] = 40000
    run(L, (24, 7), counts=counts)


@pytest.mark.parametrize("L,every", [(1, 1), (255, 3), (4097, 7), (70003, 5), (70003, 150), (300004, 1)])
@pytest.mark.parametrize("n_modes,digest", [(0, True), (2, False)])
def test_logs_within_a_launch(L, every, n_modes, digest):
    """Logs summed from the registers, at steps inside and at the end of a
    launch and of lattices with positions after their last site, equal the
    moments read between the steps."""
    import torch
    a, b = (Lattice(L, 7, rho=30.0, u0=0.1) for _ in range(2))
    g = torch.Generator(device="cuda").manual_seed(3)
    tw = torch.randint(-2**30, 2**30, (2 * n_modes * L,), dtype=torch.int32, device="cuda", generator=g) \
        if n_modes else None
    n = 6
    out, row = (torch.zeros(k * 33, dtype=torch.int64, device="cuda") for k in (n, 1))
    for l in (a, b):
        l.step(2)
    a.step_log(every, n, out, tw, n_modes, digest=digest)
    assert a.check() == 0
    torch.cuda.synchronize()
    got = out.cpu().numpy().reshape(n, 33)
    for j in range(n):
        b.step(every)
        b.moments_to_device(row, tw, n_modes, digest=digest)
        b.check()
        torch.cuda.synchronize()
        assert np.array_equal(got[j], row.cpu().numpy()), j
    assert a.moments(digest=True) == b.moments(digest=True)
    a.close()
    b.close()

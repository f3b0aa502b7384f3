"""The kernels that hold sites in registers at the sizes where each number of
sites per lane is chosen: every count equals the oracle's on long lattices whose
length is no multiple of 8, with crowded stretches that the image (built for the
mean) leaves undecided, one across the lattice's end; lattices too many for a
round of blocks; and whole states equal those of one step per launch."""
import numpy as np
import pytest

import oracle as O
import synth
from paper_1706_01094_amd.mclg import DRAIN_PATCH, Lattice

pytestmark = pytest.mark.gpu


def say(*a):
    print("[gpu]", *a, flush=True)


def crowded(L, rho, seed, stretches):
    """A Poisson start with stretches (first site, sites, counts) of equal sites."""
    rng = np.random.default_rng(seed)
    c = np.stack([rng.poisson(rho * w, L).astype(np.uint16) for w in (1 / 6, 2 / 3, 1 / 6)])
    for x, n, abc in stretches:
        c[:, np.arange(x, x + n) % L] = np.array(abc, dtype=np.uint16)[:, None]
    return c


def compare(g, o, n, what):
    for r in range(n):
        a, b = g.counts(r), o.counts(r)
        if not np.array_equal(a, b):
            bad = np.argwhere(a != b)
            raise AssertionError(f"{what}, replica {r}: {len(bad)} counts differ, first {bad[:4].tolist()}")


@pytest.mark.parametrize("L,steps,lane", [(8000003, 20, 16), (30000001, 18, 24)])
def test_long_ragged_lattices(L, steps, lane):
    say("ragged", L, steps)
    full = (60, 45, 60)
    c = crowded(L, 30.0, L, [(L - 2500, 6000, full), (L // 3, 9000, full), (L // 2, 300, (100, 100, 90)),
                             (L // 5 + 3, 40, full)])
    g = Lattice(L, 19, counts=c)
    p = g.step_plan(steps)
    assert p["sites_per_lane"] == lane and p["extra_sites"] > 0, p
    o = O.OracleSim([L], 19)
    o.init_counts(0, c)
    g.step(steps)
    o.step(steps)
    assert g.check() == 0
    compare(g, o, 1, L)
    g.close()
    o.close()


@pytest.mark.parametrize("n,L,lane", [(600, 1500, 24), (2000, 1536, 24), (300, 20000, 24)])
@pytest.mark.parametrize("stretch", [0, 150])
def test_rings_of_more_lattices_than_blocks(n, L, lane, stretch):
    """Turned copies of one start, so that all share an image."""
    say("rings", n, L, stretch)
    rng = np.random.default_rng(n)
    one = crowded(L, 30.0, n, [(L - 70, stretch, (50, 40, 55))] if stretch else [])
    c = np.stack([np.roll(one, int(k), axis=1) for k in rng.integers(0, L, n)])
    g = Lattice(np.full(n, L, dtype=np.uint64), 23, counts=c.reshape(-1))
    p = g.step_plan(12)
    assert p["sites_per_lane"] == lane and p["extra_sites"] == 0, p
    pick = [0, 1, 255, 256, n - 1] + [int(r) for r in rng.integers(0, n, 20)]
    o = O.OracleSim([L] * len(pick), 23, replica_id=pick)
    for j, r in enumerate(pick):
        o.init_counts(j, c[r])
    for k in (12, 5):
        g.step(k)
        o.step(k)
        assert g.check() == 0
        for j, r in enumerate(pick):
            assert np.array_equal(g.counts(r), o.counts(j)), (r, k)
    g.close()
    o.close()


@pytest.mark.parametrize("L", [4096, 65536, 70003, 1000003, (1 << 22) + 5, 1 << 24, 30000001])
def test_same_as_one_step_per_launch(L):
    a, b = (Lattice(L, 29, rho=50.0, u0=0.1) for _ in range(2))
    b.set_drain(1)
    for n in (3, 40, 100):
        say(L, n, a.step_plan(n))
        assert a.step_plan(n)["sites_per_lane"] > 0 and b.step_plan(n)["sites_per_lane"] == 0
        a.step(n)
        b.step(n)
        assert a.moments(digest=True) == b.moments(digest=True)
    a.close()
    b.close()


def test_batch_same_as_one_step_per_launch():
    """The 1024 replicas, with the draws of a chunk resolved before its store."""
    man = synth.replica_manifest()
    a, b = (Lattice(man["L"], synth.BATCHED["seed"], rho=man["rho"], u0=man["u0"], replica_id=man["replica_id"])
            for _ in range(2))
    b.set_drain(DRAIN_PATCH)
    assert a.step_plan(50)["sites_per_lane"] > 0 and b.step_plan(50)["sites_per_lane"] == 0
    a.step(50)
    b.step(50)
    assert a.moments(digest=True) == b.moments(digest=True)
    a.close()
    b.close()

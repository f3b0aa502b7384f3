"""The three forms of the D2Q9 rules (sums in bytes, in halves, and for any N
and D) at the sizes where one takes over from the next, with draws that are
rejected often, and with a block that goes from one to the next: every count
equals the oracle's."""
import numpy as np
import pytest

from paper_1706_01094_amd.mclg import LAMBDA9_PAPER
from tests.test_gpu_d2q9 import pair9, same9

pytestmark = pytest.mark.gpu

# D = 147456 with weights that are multiples of 9; the largest D of the packed
# tables; one past it; a quarter of the target draws rejected, few weights and
# many
LAMS = {"paper": LAMBDA9_PAPER, "2^15": [(1, 256)] * 9, "2^16": [(1, 512)] * 9,
        "rejected": [(3 << 20, 3 << 22)] * 9, "rejected wide": [(2000003, 12582917)] * 9}


def spread(N, rng):
    """N particles over nine velocities."""
    return rng.multinomial(N, np.full(9, 1 / 9)).astype(np.uint16)


@pytest.mark.parametrize("lams", list(LAMS))
@pytest.mark.parametrize("top", [127, 128, 32767, 32768, 60000])
def test_largest_site_at_the_edge_of_a_table(lams, top):
    rng = np.random.default_rng(top)
    Ly, Lx = 9, 60
    c = np.zeros((9, Ly, Lx), dtype=np.uint16)
    for s in range(Lx * Ly):
        N = [0, 1, 2, 20, min(top, 100)][s % 5]
        c[:, s // Lx, s % Lx] = spread(N, rng)
    c[:, 4, 31] = spread(top, rng)
    g, o = pair9(Lx, Ly, 5, lams=LAMS[lams], counts=c.reshape(-1))
    for _ in range(4):
        g.step(1)
        assert o.step(1) == 0
        same9(g, o, 1)
    g.close()


def test_blocks_that_change_tables():
    """More tiles than blocks: the tiles that a block takes second hold sites
    for the half table, one of them for the wide one."""
    rng = np.random.default_rng(1)
    Ly, Lx = 1433, 1500
    c = rng.integers(0, 5, size=(9, Ly * Lx)).astype(np.uint16)
    late = np.arange(8192 * 256 + 100, Ly * Lx, 700)
    c[:, late] += 30
    c[:, 8192 * 256 + 300] = 5000
    g, o = pair9(Lx, Ly, 6, counts=c.reshape(-1))
    g.step(2)
    assert o.step(2) == 0
    same9(g, o, 1)
    g.close()


@pytest.mark.parametrize("Lx,Ly", [(1, 1), (1, 7), (2, 2), (64, 1), (13, 5), (32, 16), (27, 19), (31, 33)])
def test_several_steps_in_a_launch(Lx, Ly):
    """Lattices of up to 512 sites (and some more), whole in a block's LDS: sites that need
    each of the tables, empty ones, and lengths of one row or column."""
    rng = np.random.default_rng(Lx)
    n = [Lx, max(1, Lx - 1), 3]
    rows = []
    for lx in n:
        c = rng.integers(0, 9, size=(9, Ly * lx)).astype(np.uint16)
        c[:, ::5] = 0
        c[:, 0] += 40
        rows.append(c.reshape(-1))
    g, o = pair9(n, [Ly] * 3, 8, counts=np.concatenate(rows))
    for k in (20, 6, 17):
        g.step(k)
        assert o.step(k) == 0
        same9(g, o, 3)
    g.close()
    c = np.zeros((9, Ly, Lx), dtype=np.uint16)
    c[:] = 3
    c[:, 0, 0] = 4000
    g, o = pair9(Lx, Ly, 8, counts=c.reshape(-1))
    g.step(18)
    assert o.step(18) == 0
    same9(g, o, 1)
    g.close()

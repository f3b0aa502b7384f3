"""D2Q9 lattices without sub-collisions (C = 0): a step changes no count, but a
site that does not fit 16 bits is still reported, by one step per launch and by
several."""
import numpy as np
import pytest

from paper_1706_01094_amd.mclg import E_RANGE
from tests.test_gpu_d2q9 import pair9

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("C", [0, 2])
@pytest.mark.parametrize("Lx,Ly", [(16, 16), (40, 30)])
@pytest.mark.parametrize("n", [1, 5])
def test_overflow_is_flagged_and_kept(C, Lx, Ly, n):
    c = np.full((9, Ly, Lx), 2, dtype=np.uint16)
    g, o = pair9(Lx, Ly, 4, C=C, counts=c.reshape(-1))
    g.step(n)
    assert o.step(n) == 0 and g.check() == 0
    g.close()
    c[:, Ly // 2, Lx // 3] = 8000
    g, o = pair9(Lx, Ly, 4, C=C, counts=c.reshape(-1))
    g.step(n)
    assert o.step(n) == E_RANGE and g.check() == E_RANGE
    assert np.array_equal(g.counts(0, allow_range=True), o.counts(0))
    g.close()

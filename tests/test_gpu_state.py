"""State transfers (qnsch_set_state, qnsch_get_state): fields come back
bitwise, faces on walls as zero, NULL fields as zero also after another
state."""
import numpy as np
import pytest

from paper_1703_06606_amd import qnsch as Q
from paper_1703_06606_amd import workloads as W

FIELDS = ("c", "mu", "p", "u", "v")


@pytest.mark.gpu
@pytest.mark.parametrize("precision", [Q.FP64, Q.MIXED])
@pytest.mark.parametrize("m1,m2", [(4, 4), (40, 24), (8, 264), (264, 8)])
@pytest.mark.parametrize("bcx,bcy", [(0, 0), (1, 0), (0, 1), (1, 1)])
def test_state_round_trip(m1, m2, bcx, bcy, precision):
    grid = dict(m1=m1, m2=m2, Lx=1.0, Ly=m2 / m1, bcx=bcx, bcy=bcy, levels=0)
    s = Q.Solver(grid, W.params(1.0, 3.0, 1.0, 1.0, Re=100.0, We=100.0, inv_Fr=0.0, eps=0.05),
                 dict(W.default_opts(), precision=precision))
    rng = np.random.default_rng(m1 + m2 + bcx)
    w = {k: rng.uniform(-1, 1, (m2, m1)) for k in FIELDS}
    s.set_state(*[w[k] for k in FIELDS])
    if not bcx:
        w["u"][:, 0] = 0.0
    if not bcy:
        w["v"][0] = 0.0
    got = s.get_state()
    for k in FIELDS:
        assert np.array_equal(got[k], w[k]), k
    s.set_state(w["c"], u=w["u"])
    got = s.get_state()
    assert np.array_equal(got["c"], w["c"]) and np.array_equal(got["u"], w["u"])
    for k in ("mu", "p", "v"):
        assert not got[k].any(), k

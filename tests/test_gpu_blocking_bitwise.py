"""Fused sweeps (one or two per launch), half-sweeps and the folded coarse-grid
correction share their arithmetic, contracted within an expression only: two
steps end bitwise the same with any blocking."""
import numpy as np
import pytest

from paper_1703_06606_amd import qnsch as Q
from paper_1703_06606_amd import workloads as W

FIELDS = ("c", "mu", "p", "u", "v")
KINDS = {"coupled": {}, "segregated": dict(smoother=W.SMOOTH_SEGREGATED), "projection": dict(scheme=Q.PROJECTION),
         "mixed": dict(precision=Q.MIXED)}


@pytest.mark.gpu
@pytest.mark.parametrize("kind", list(KINDS))
@pytest.mark.parametrize("m1,m2,bcx,nu1,nu2", [
    (40, 24, 0, 2, 2),    # ragged tiles
    (64, 64, 1, 3, 2),    # a periodic axis, an odd last sweep
    (64, 128, 0, 4, 4),   # several two-sweep launches
    (160, 128, 0, 2, 2),  # more 8 x 8 tiles than compute units: one sweep per launch
])
def test_blocking_does_not_change_a_bit(m1, m2, bcx, nu1, nu2, kind):
    cfg = W.rising_drop(m1, m2, eps=0.06, radius=0.2)
    grid = dict(m1=m1, m2=m2, Lx=1.0, Ly=m2 / m1, bcx=bcx, bcy=0, levels=0)
    states = []
    for blocking in (0, 1, 2):
        opts = dict(W.default_opts(1e-8), blocking=blocking, nu1=nu1, nu2=nu2, **KINDS[kind])
        s = Q.Solver(grid, cfg["params"], opts)
        s.set_state(cfg["state"]["c"])
        for _ in range(2):
            assert s.step(cfg["dt"]) == Q.OK
        states.append(s.get_state())
    for w in states[1:]:
        for k in FIELDS:
            assert np.array_equal(w[k], states[0][k]), (k, np.abs(w[k] - states[0][k]).max())

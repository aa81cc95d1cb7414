"""Levels whose periodic axis is long enough for two sweeps in a launch but not
for one (16 cells), with sweep counts that do not pair: FP64 cycles against
the oracle's (1e-10 of the field's maximum, the parity bound), mixed precision
against the oracle's converged step (1e-6, the mixed-precision bound)."""
import numpy as np
import pytest

import oracle as OR
from paper_1703_06606_amd import qnsch as Q
from paper_1703_06606_amd import workloads as W

FIELDS = ("c", "mu", "p", "u", "v")


def rel(a, b, floor=1e-9):
    return np.abs(a - b).max() / max(np.abs(b).max(), floor)


@pytest.mark.gpu
@pytest.mark.parametrize("precision", [Q.FP64, Q.MIXED])
@pytest.mark.parametrize("m1,m2,bcx,bcy", [(16, 16, 1, 1), (16, 64, 1, 0), (64, 16, 0, 1)])
@pytest.mark.parametrize("nu1,nu2", [(2, 4), (4, 2), (3, 2)])
def test_cycles_match_oracle(m1, m2, bcx, bcy, nu1, nu2, precision):
    cfg = W.rising_drop(m1, m2, eps=0.06, radius=0.2)
    x = (np.arange(m1) + 0.5) / m1
    y = ((np.arange(m2) + 0.5) / m1)[:, None]
    d = np.hypot(np.sin(np.pi * (x - 0.45)) / np.pi, np.sin(np.pi * m1 / m2 * (y - 0.4 * m2 / m1)) * m2 / m1 / np.pi)
    c = 0.5 * (1.0 + np.tanh((d - 0.2) / (2 * np.sqrt(2) * 0.06)))
    grid = dict(m1=m1, m2=m2, Lx=1.0, Ly=m2 / m1, bcx=bcx, bcy=bcy, levels=0)
    par = dict(cfg["params"], inv_Fr=0.0)
    opts = dict(W.default_opts(1e-10), blocking=2, nu1=nu1, nu2=nu2)
    o = OR.Oracle(grid, par, opts)
    s = Q.Solver(grid, par, dict(opts, precision=precision))
    for z in (s, o):
        z.set_state(c)
    if precision == Q.MIXED:
        assert o.step(cfg["dt"]) == OR.OK
        assert s.step(cfg["dt"]) == Q.OK
        a, r = s.get_state(), o.get_state()
        for k in FIELDS:
            assert rel(a[k], r[k]) < 1e-6, (k, rel(a[k], r[k]))
        return
    for z in (s, o):
        z.begin_step(cfg["dt"])
    for it in range(2):
        for z in (s, o):
            z.vcycle()
        a, r = s.get_state(), o.get_state()
        for k in FIELDS:
            assert rel(a[k], r[k]) < 1e-10, (it, k, rel(a[k], r[k]))

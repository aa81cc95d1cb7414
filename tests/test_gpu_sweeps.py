"""Two sweeps per launch on 8 x 8 tiles, and the bottom levels of a cycle in
one workgroup, at the sizes where they can go wrong: ragged tiles, the shortest
periodic axis that a widened tile wraps once, the largest level that takes two
sweeps a launch and the first that does not, sweep counts that leave the cell
unknowns in either set, a periodic axis of two cells and more cells of a colour
than one pass of a workgroup takes.  FP64 against the oracle's cycles (1e-10
of the field's maximum, the parity bound), mixed precision against the oracle's
converged step (1e-6, the mixed-precision bound)."""
import numpy as np
import pytest

import oracle as OR
from paper_1703_06606_amd import qnsch as Q
from paper_1703_06606_amd import workloads as W

FIELDS = ("c", "mu", "p", "u", "v")


def rel(a, b, floor=1e-9):
    return np.abs(a - b).max() / max(np.abs(b).max(), floor)


def _cfg(m1, m2, bcx, bcy):
    cfg = W.rising_drop(m1, m2, eps=0.06, radius=0.2)
    cfg["grid"] = dict(m1=m1, m2=m2, Lx=1.0, Ly=m2 / m1, bcx=bcx, bcy=bcy, levels=0)
    x = (np.arange(m1) + 0.5) / m1
    y = ((np.arange(m2) + 0.5) / m1)[:, None]
    d = np.hypot(np.sin(np.pi * (x - 0.45)) / np.pi, np.sin(np.pi * m1 / m2 * (y - 0.4 * m2 / m1)) * m2 / m1 / np.pi)
    cfg["state"]["c"] = 0.5 * (1.0 + np.tanh((d - 0.2) / (2 * np.sqrt(2) * 0.06)))
    if bcx or bcy:
        cfg["params"] = dict(cfg["params"], inv_Fr=0.0)
    return cfg


@pytest.mark.gpu
@pytest.mark.parametrize("kind", ["coupled", "segregated", "projection", "mixed"])
@pytest.mark.parametrize("m1,m2,bcx,bcy,nu1,nu2", [
    (16, 16, 1, 1, 2, 2),
    (20, 36, 0, 0, 2, 2),
    (36, 20, 1, 0, 2, 4),
    (40, 24, 0, 1, 4, 2),
    (24, 40, 0, 0, 4, 4),
    (24, 24, 1, 0, 1, 1),
    (24, 24, 0, 1, 3, 2),
    (12, 24, 1, 0, 2, 2),
    (128, 128, 0, 0, 2, 2),
    (160, 128, 0, 1, 2, 2),
    (16, 4, 0, 1, 2, 2),
    (8, 64, 0, 0, 2, 2),
    (64, 64, 1, 0, 2, 2),
])
def test_cycles_match_oracle(m1, m2, bcx, bcy, nu1, nu2, kind):
    cfg = _cfg(m1, m2, bcx, bcy)
    opts = dict(W.default_opts(1e-10), blocking=2, nu1=nu1, nu2=nu2)
    if kind == "segregated":
        opts["smoother"] = W.SMOOTH_SEGREGATED
    if kind == "projection":
        opts["scheme"] = Q.PROJECTION
    o = OR.Oracle(cfg["grid"], cfg["params"], opts)
    s = Q.Solver(cfg["grid"], cfg["params"], dict(opts, precision=Q.MIXED) if kind == "mixed" else opts)
    for x in (s, o):
        x.set_state(cfg["state"]["c"])
    if kind == "mixed":
        assert o.step(cfg["dt"]) == OR.OK
        assert s.step(cfg["dt"]) == Q.OK
        a, r = s.get_state(), o.get_state()
        for k in FIELDS:
            assert rel(a[k], r[k]) < 1e-6, (k, rel(a[k], r[k]))
        return
    for x in (s, o):
        x.begin_step(cfg["dt"])
    for it in range(2):
        for x in (s, o):
            x.vcycle()
        a, r = s.get_state(), o.get_state()
        for k in FIELDS:
            assert rel(a[k], r[k]) < 1e-10, (it, k, rel(a[k], r[k]))

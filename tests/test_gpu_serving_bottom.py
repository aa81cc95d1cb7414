"""Many equal requests in one server, so that every launch of the bottom levels
of a cycle is a list of several one-workgroup items: each result bit-identical
to the request run alone."""
import numpy as np
import pytest

from paper_1703_06606_amd import qnsch as Q
from paper_1703_06606_amd import workloads as W

FIELDS = ("c", "mu", "p", "u", "v")


@pytest.mark.gpu
@pytest.mark.parametrize("precision", [Q.FP64, Q.MIXED])
@pytest.mark.parametrize("lanes,requests", [(1, 12), (3, 24)])
def test_equal_requests_equal_alone(lanes, requests, precision):
    cfg = W.rising_drop(64, 128, eps=0.02)
    opts = dict(W.default_opts(1e-8), blocking=0, accel=0, precision=precision)
    nsteps = 2
    g = Q.Solver(cfg["grid"], cfg["params"], opts)
    g.set_state(cfg["state"]["c"])
    mass = []
    for _ in range(nsteps):
        assert g.step(cfg["dt"]) == Q.OK
        mass.append(g.mass())
    ref = g.get_state()
    srv = Q.Server(hbm_budget=8 << 30, max_slots=requests, lanes=lanes)
    ids = [srv.submit(cfg["grid"], cfg["params"], opts, cfg["state"]["c"], nsteps, cfg["dt"]) for _ in range(requests)]
    for _ in range(100000):
        if srv.progress(64) == 0:
            break
    for rid in ids:
        r = srv.result(rid)
        assert r["status"] == Q.OK
        for k in FIELDS:
            assert np.array_equal(r[k], ref[k]), (rid, k, np.abs(r[k] - ref[k]).max())
        assert np.array_equal(r["mass"], np.array(mass)), rid

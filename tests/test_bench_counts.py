"""Counts that bench.py derives from a run's launches (CPU only), worked out by
hand."""
import pytest

import bench as B

CELLS = [2048, 512, 128, 32]  # a 32 x 64 grid's levels


@pytest.mark.parametrize("nu1,nu2,per_cycle", [(2, 2, 2), (4, 4, 4), (2, 4, 2), (6, 2, 4)])
def test_two_sweep_launch_bytes(nu1, nu2, per_cycle):
    """A launch does two sweeps whatever nu1 and nu2 are, 104 B per cell each on
    the finest level (no right-hand sides) and 144 on coarser ones, and one
    launch of a cycle takes the prolongation (100 B per cell)."""
    opts = {"nu1": nu1, "nu2": nu2, "nu_coarse": 0, "accel": 2, "scheme": 0}
    cycles = 3
    assert B.class_bytes("smooth", 0, cycles * per_cycle, CELLS, opts) == cycles * (per_cycle * 208.0 + 100.0) * 2048
    assert B.class_bytes("smooth", 1, cycles * per_cycle, CELLS, opts) == cycles * (per_cycle * 288.0 + 100.0) * 512

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


def test_kernels_of_a_reduction():
    """more than 512 partials are folded first: 512 x 2048 has 4096 tiles, 256 x
    512 exactly 512; 16 x 8208 has 513 of both kinds, 8 x 8200 513 tiles but 257
    blocks of 256 cells"""
    for op in ("residual", "residual0", "residual_acc", "step_end", "dissipation", "diagnostics"):
        assert B.kernels_of_op(op, 256, 512) == 2
        assert B.kernels_of_op(op, 512, 2048) == 3
        assert B.kernels_of_op(op, 16, 8208) == 3
    assert B.kernels_of_op("residual_acc", 8, 8200) == 3 and B.kernels_of_op("step_end", 8, 8200) == 2
    for op in ("halfsweep", "smooth", "coarse_solve", "accelerate"):
        assert B.kernels_of_op(op, 512, 2048) == 1

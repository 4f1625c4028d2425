"""hilore_allocate where rows have no padding cells (N_B + 1 a multiple of 64), with
odd unit counts and with values of every kind behind actions that are not available.

The DP reads those actions as -inf and ignores their utilities, whatever they are;
results must equal the oracle's bit for bit.
"""
import numpy as np
import pytest

from paper_2609_33570_amd import workloads as wl
from test_gpu_alloc import assert_same, gpu_allocate, oracle_allocate

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("grid", [(63, 63), (127, 40), (62, 1), (255, 255), (1023, 300)])
@pytest.mark.parametrize("U", [1, 2, 3, 8, 33])
def test_unpadded_rows(hl, orc, grid, U):
    inst = wl.alloc_small(U, seed=7000 + U + grid[0], scale=32.0)
    assert_same(gpu_allocate(hl, inst, *grid), oracle_allocate(orc, inst, *grid), f"U={U} {grid}")


@pytest.mark.parametrize("bad", [float("nan"), float("inf"), -float("inf"), -1.0, 0.0])
def test_unavailable_actions(hl, orc, bad):
    base = wl.alloc_small(21, seed=77, scale=16.0)
    third = np.arange(21) % 3
    tau_h = np.where(third == 0, bad, base.tau_h)
    tau_l = np.where(third == 1, bad, base.tau_l)
    psi = np.where(third == 2, bad if bad != 0.0 else np.inf, base.psi)
    inst = wl.AllocInstance(base.q, base.verified, tau_h, tau_l, base.dm_h, base.dm_l, psi,
                            base.m_res, base.delta_b)
    for grid in ((63, 63), (200, 77)):
        assert_same(gpu_allocate(hl, inst, *grid), oracle_allocate(orc, inst, *grid), f"{bad} {grid}")

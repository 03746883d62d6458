"""The Korteweg diagnostic of lattices with moving walls: its phase field is the one
of the state's own densities.

Tolerance: both are quotients of 19-term sums, FP64 1e-12 and FP32 (and the FP32
arithmetic of 16-bit storage) 5e-6: 38 roundings of 6e-8 and the division.
"""
import numpy as np
import pytest

from paper_2005_12764_amd import lb
from paper_2005_12764_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage", [W.F64, W.F32, W.F16])
def test_phase_blocks_follow_the_densities(storage):
    nx, ny, nz = 66, 12, 20
    rr, rb, u = W.random_state(41, (nz, ny, nx))
    p = W.base_params(nx, ny, nz, bc=(0, 1, 1), storage=storage, tau_r=0.8, tau_b=0.8, A=0.01)
    p["wall_velocity"] = ((0, 0, 0),) * 4 + ((-0.01, 0, 0), (0.01, 0, 0))
    with lb.Lattice(p) as L:
        L.init(rr, rb, u).step(4)
        _, phi = L.korteweg(0.05, 2)
        a, b, _ = L.moments()
    ref = ((a - b) / (a + b)).reshape(nz // 2, 2, ny // 2, 2, nx // 2, 2).mean((1, 3, 5))
    assert np.abs(phi - ref).max() <= (1e-12 if storage == W.F64 else 5e-6)

"""The Korteweg tensor and phase blocks of lattices with moving walls against the
oracle, on walls of each axis and for every block size.

Tolerances: the phase field agrees as the parity tests' populations do (FP64
1e-12, FP32 1e-5, fp16 2e-4, bf16 2e-3).  With |phi| <= 1 the stencils give |Lap|
<= 8 and |grad_a| <= 1, their errors at most 8 and 1 times the field's e, so K is
off by at most lam (16 + 3 + 2) e; block means add nothing.
"""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2005_12764_amd import lb
from paper_2005_12764_amd import workloads as W
from tests.helpers import oracle_params

pytestmark = pytest.mark.gpu

TOL = {W.F64: 1e-12, W.F32: 1e-5, W.F16: 2e-4, W.BF16: 2e-3}
MOVING = ((0, 0.004, -0.002), (0, -0.003, 0.002), (0.005, 0, 0.001), (-0.004, 0, 0.003), (-0.01, 0.002, 0),
          (0.01, -0.001, 0))
LAM = 0.05


@pytest.mark.parametrize("n,bc", [((72, 16, 24), (0, 1, 1)), ((24, 16, 8), (1, 0, 1)), ((40, 24, 16), (0, 0, 1)),
                                  ((64, 8, 40), (1, 1, 1))], ids=["yz", "xz", "z", "xyz"])
@pytest.mark.parametrize("storage", [W.F64, W.F32, W.F16, W.BF16])
def test_tensor_between_moving_walls(storage, n, bc):
    nx, ny, nz = n
    rr, rb, u = W.random_state(43, (nz, ny, nx))
    p = W.base_params(nx, ny, nz, bc=bc, storage=storage, tau_r=0.8, tau_b=1.1, A=0.01)
    p["wall_velocity"] = MOVING
    with lb.Lattice(p) as L:
        L.init(rr, rb, u).step(5)
        blocks = {b: L.korteweg(LAM, b) for b in (1, 2, 4, 8)}
    prm = oracle_params(p)
    phi = O.phase_field(prm, O.step(prm, O.init(prm, rr, rb, u), 5))
    K = O.korteweg(prm, phi, LAM)
    for b, (k, f) in blocks.items():
        assert np.abs(f - O.block_average(prm, phi, b)).max() <= TOL[storage], b
        assert np.abs(k - O.block_average(prm, K, b)).max() <= 21 * LAM * TOL[storage], b

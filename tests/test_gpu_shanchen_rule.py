"""Shan-Chen steps on both sides of the rule between one pass and two (FP32: chunks of
three planes or more, two of full rows, and 0.53 of the lanes take one), and the short chunks of two
passes, against the oracle.

Tolerances: the parity tests' (FP64 1e-12, FP32 1e-5 relative L2).
"""
import pytest

from oracle import oracle as O
from paper_2005_12764_amd import lb
from paper_2005_12764_amd import workloads as W
from tests.helpers import oracle_params, state_errors

pytestmark = pytest.mark.gpu

TOL = {W.F64: 1e-12, W.F32: 1e-5}
ONE = [(100, 63, 50), (64, 60, 97), (130, 33, 90), (34, 65, 130), (64, 60, 63)]  # chunks of 4, 4, 6, 5 and 2 planes
TWO = [(64, 60, 31), (33, 65, 130), (100, 63, 32), (24, 40, 30)]        # 1 or 2 planes, or few lanes


@pytest.mark.parametrize("bc", [(0, 0, 0), (0, 1, 1), (1, 0, 1)], ids=["periodic", "yz", "xz"])
@pytest.mark.parametrize("n", ONE + TWO, ids=str)
@pytest.mark.parametrize("storage", [W.F64, W.F32])
def test_either_side_of_the_rule(storage, n, bc):
    nx, ny, nz = n
    rr, rb, u = W.random_state(67, (nz, ny, nx))
    p = W.base_params(nx, ny, nz, bc=bc, storage=storage, tau_r=1.0, tau_b=1.0, body_force=(1e-5, -2e-6, 3e-6))
    p.update(model=lb.MODEL_SHAN_CHEN, g_sc=0.2, A=0.0)
    with lb.Lattice(p) as L:
        f = L.init(rr, rb, u).step(4).state()
    prm = oracle_params(p)
    assert state_errors(f, O.step(prm, O.init(prm, rr, rb, u), 4))["worst"] <= TOL[storage]

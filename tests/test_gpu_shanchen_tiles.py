"""The one-pass Shan-Chen step at row, column and chunk remainders, periodic and
between resting walls, and the two passes of FP64 at the chunk lengths of small
lattices, against the oracle.

Tolerances: the parity tests' (FP64 1e-12, FP32 1e-5 relative L2).
"""
import pytest

from oracle import oracle as O
from paper_2005_12764_amd import lb
from paper_2005_12764_amd import workloads as W
from tests.helpers import oracle_params, state_errors

pytestmark = pytest.mark.gpu

TOL = {W.F64: 1e-12, W.F32: 1e-5}


@pytest.mark.parametrize("n,bc", [((65, 9, 5), (0, 0, 0)), ((64, 8, 33), (0, 1, 1)), ((3, 17, 2), (1, 0, 0)),
                                  ((130, 7, 4), (1, 1, 1)), ((5, 1, 1), (0, 0, 0))],
                         ids=["remainders", "walls_yz", "narrow", "walls", "row"])
@pytest.mark.parametrize("storage", [W.F64, W.F32])
def test_edges_against_the_oracle(storage, n, bc):
    nx, ny, nz = n
    rr, rb, u = W.random_state(37, (nz, ny, nx))
    p = W.base_params(nx, ny, nz, bc=bc, storage=storage, tau_r=1.0, tau_b=1.0, body_force=(1e-5, -2e-6, 3e-6))
    p.update(model=lb.MODEL_SHAN_CHEN, g_sc=0.2, A=0.0)
    with lb.Lattice(p) as L:
        f = L.init(rr, rb, u).step(6).state()
    prm = oracle_params(p)
    e = state_errors(f, O.step(prm, O.init(prm, rr, rb, u), 6))
    assert e["worst"] <= TOL[storage], e

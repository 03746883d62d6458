"""The automatic choice of lattices with walls: FP32 between walls at rest takes
16-row tiles by itself.

Tolerance: the parity tests' (FP32 1e-5 relative L2).
"""
import pytest

from oracle import oracle as O
from paper_2005_12764_amd import lb
from paper_2005_12764_amd import workloads as W
from tests.helpers import oracle_params, state_errors

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bc", [(0, 1, 1), (1, 1, 1), (1, 0, 0)], ids=["yz", "xyz", "x"])
def test_fp32_between_walls_at_rest(bc):
    nx, ny, nz = 191, 95, 66                          # its choice is 16 rows
    rr, rb, u = W.random_state(61, (nz, ny, nx))
    p = W.base_params(nx, ny, nz, bc=bc, storage=W.F32, tau_r=0.7, tau_b=1.2, A=0.01, body_force=(1e-5, 0, 0))
    with lb.Lattice(p) as L:
        f = L.init(rr, rb, u).step(3).state()
    prm = oracle_params(p)
    assert state_errors(f, O.step(prm, O.init(prm, rr, rb, u), 3))["worst"] <= 1e-5

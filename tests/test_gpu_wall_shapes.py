"""The automatic choice of lattices with walls: FP64 between moving walls with the
widest probe halo steps in two passes where tiles fill few lanes and with one read
where they fill them; FP32 between walls at rest takes 16-row tiles by itself.

Tolerances: the parity tests' (FP64 1e-12, FP32 1e-5 relative L2).
"""
import pytest

from oracle import oracle as O
from paper_2005_12764_amd import lb
from paper_2005_12764_amd import workloads as W
from tests.helpers import oracle_params, state_errors

pytestmark = pytest.mark.gpu

MOVING = ((0, 0.004, -0.002), (0, -0.003, 0.002), (0.005, 0, 0.001), (-0.004, 0, 0.003), (-0.01, 0.002, 0),
          (0.01, -0.001, 0))


@pytest.mark.parametrize("nx,K,kernel", [(30, 4, lb.KERNEL_TWOPASS), (57, 4, lb.KERNEL_TWOPASS), (58, 4, lb.KERNEL_FUSED),
                                         (64, 4, lb.KERNEL_FUSED), (30, 3, lb.KERNEL_FUSED)])
@pytest.mark.parametrize("bc", [(0, 1, 1), (1, 0, 1)], ids=["yz", "xz"])
def test_fp64_between_moving_walls(bc, nx, K, kernel):
    ny, nz = 14, 12
    rr, rb, u = W.random_state(59, (nz, ny, nx))
    p = W.base_params(nx, ny, nz, bc=bc, storage=W.F64, tau_r=0.7, tau_b=1.2, A=0.01, nc_strength=0.01, nc_range=K)
    p["wall_velocity"] = MOVING
    with lb.Lattice(p) as L:
        assert L.kernel == kernel
        f = L.init(rr, rb, u).step(5).state()
    prm = oracle_params(p)
    assert state_errors(f, O.step(prm, O.init(prm, rr, rb, u), 5))["worst"] <= 1e-12


@pytest.mark.parametrize("bc", [(0, 1, 1), (1, 1, 1), (1, 0, 0)], ids=["yz", "xyz", "x"])
def test_fp32_between_walls_at_rest(bc):
    nx, ny, nz = 191, 95, 66                          # its choice is 16 rows
    rr, rb, u = W.random_state(61, (nz, ny, nx))
    p = W.base_params(nx, ny, nz, bc=bc, storage=W.F32, tau_r=0.7, tau_b=1.2, A=0.01, body_force=(1e-5, 0, 0))
    with lb.Lattice(p) as L:
        f = L.init(rr, rb, u).step(3).state()
    prm = oracle_params(p)
    assert state_errors(f, O.step(prm, O.init(prm, rr, rb, u), 3))["worst"] <= 1e-5

"""Moments, export and totals of packed and 16-bit states, whose kernels march
z-chunks of 16 or more planes with the source records in LDS: chunk, row and
column remainders, walls at rest and moving, against the oracle and against sums
of the exported state.

Tolerances: the parity tests' against the oracle (FP64 1e-12, FP32 1e-5, fp16
2e-4, bf16 2e-3).  Moments against sums of the exported values: 19 additions of
values below 1 in the storage's arithmetic, 19 eps/2 (FP64 2e-15, FP32 1.2e-6).
Totals are FP64 sums of the exported values: 1e-13 relative, 1e-12 on momenta
(not on moving walls: there the export adds the wall terms in FP64 and the totals
in the storage's arithmetic, both site by site).
"""
import math

import numpy as np
import pytest

from oracle import oracle as O
from paper_2005_12764_amd import lb
from paper_2005_12764_amd import workloads as W
from tests.helpers import oracle_params, state_errors

pytestmark = pytest.mark.gpu

TOL = {W.F64: 1e-12, W.F32: 1e-5, W.F16: 2e-4, W.BF16: 2e-3}
MOVING = ((0, 0.004, -0.002), (0, -0.003, 0.002), (0.005, 0, 0.001), (-0.004, 0, 0.003), (-0.01, 0.002, 0),
          (0.01, -0.001, 0))


@pytest.mark.parametrize("n,bc,moving", [((65, 17, 35), (0, 0, 0), False), ((64, 9, 33), (0, 1, 1), False),
                                         ((130, 7, 18), (1, 0, 0), False), ((66, 8, 17), (1, 1, 1), True),
                                         ((3, 33, 2), (0, 0, 0), False)],
                         ids=["remainders", "walls_yz", "walls_x", "moving", "narrow"])
@pytest.mark.parametrize("storage", [W.F64, W.F32, W.F16, W.BF16])
def test_readings_of_a_stepped_state(storage, n, bc, moving):
    nx, ny, nz = n
    rr, rb, u = W.random_state(29, (nz, ny, nx))
    p = W.base_params(nx, ny, nz, bc=bc, storage=storage, tau_r=0.7, tau_b=1.2, A=0.01, body_force=(1e-5, -2e-6, 3e-6))
    if moving:
        p["wall_velocity"] = MOVING
    with lb.Lattice(dict(p, kernel=lb.KERNEL_FUSED)) as L:
        L.init(rr, rb, u).step(4)
        f, (mr, mb, mj), t = L.state(), L.moments(), L.totals()
        if storage in (W.F64, W.F32):
            # the same values in pair arrays, through the per-site kernels
            L.load_raw(L.save_raw())
            assert np.array_equal(L.state(), f)
            again = L.moments()
            assert all(np.array_equal(a, b) for a, b in zip(again, (mr, mb, mj)))
    prm = oracle_params(p)
    e = state_errors(f, O.step(prm, O.init(prm, rr, rb, u), 4))
    assert e["worst"] <= TOL[storage], e
    c, _, _, _ = O.tables()
    j = np.einsum("kixyz,ia->axyz", f, c.astype(float))
    eps = 2e-15 if storage == W.F64 else 1.2e-6
    for a, b in ((mr, f[0].sum(0)), (mb, f[1].sum(0)), (mj, j)):
        assert np.abs(a - b).max() <= eps * max(1.0, np.abs(b).max())
    tot = t[:, 0] + t[:, 1]
    assert tot[6] == 0.0
    if moving:
        return
    assert math.isclose(tot[0], math.fsum(f[0].ravel()), rel_tol=1e-13)
    assert math.isclose(tot[1], math.fsum(f[1].ravel()), rel_tol=1e-13)
    for a in range(3):
        assert abs(tot[2 + a] - math.fsum(j[a].ravel())) < 1e-12

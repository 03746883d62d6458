"""Row counts of the one-read tile that a storage takes by itself: 12 rows in 16
bits and 16 in FP32, at row, column and chunk remainders, with the near-contact
halo and without, against the oracle.

Tolerances: the parity tests' (FP32 1e-5, fp16 2e-4, bf16 2e-3 relative L2).
"""
import pytest

from oracle import oracle as O
from paper_2005_12764_amd import lb
from paper_2005_12764_amd import workloads as W
from tests.helpers import oracle_params, state_errors

pytestmark = pytest.mark.gpu

TOL = {W.F32: 1e-5, W.F16: 2e-4, W.BF16: 2e-3}


@pytest.mark.parametrize("n,bc", [((65, 25, 5), (0, 0, 0)), ((64, 11, 4), (0, 1, 1)), ((70, 12, 3), (1, 0, 0))],
                         ids=["remainders", "walls_yz", "walls_x"])
@pytest.mark.parametrize("storage,rows", [(W.F32, 16), (W.F16, 12), (W.BF16, 12)])
def test_rows_at_the_edges_of_a_lattice(storage, rows, n, bc, monkeypatch):
    nx, ny, nz = n
    rr, rb, u = W.random_state(31, (nz, ny, nx))
    p = W.base_params(nx, ny, nz, bc=bc, storage=storage, tau_r=0.7, tau_b=1.2, A=0.01, body_force=(1e-5, -2e-6, 3e-6))
    monkeypatch.setenv("LB_SINGLE_TY", str(rows))
    monkeypatch.setenv("LB_TZ", "2")
    with lb.Lattice(dict(p, kernel=lb.KERNEL_FUSED)) as L:
        f = L.init(rr, rb, u).step(9).state()
    prm = oracle_params(p)
    e = state_errors(f, O.step(prm, O.init(prm, rr, rb, u), 9))
    assert e["worst"] <= TOL[storage], e


@pytest.mark.parametrize("storage,rows", [(W.F32, 16), (W.F16, 12)])
def test_rows_with_the_near_contact_halo(storage, rows, monkeypatch):
    w = W.single_droplet(seed=5, storage=storage)
    p = dict(w.params, nc_strength=0.01, nc_range=2)
    monkeypatch.setenv("LB_SINGLE_TY", str(rows))
    monkeypatch.setenv("LB_TZ", "5")
    with lb.Lattice(dict(p, kernel=lb.KERNEL_FUSED)) as L:
        f = L.init(w.rho_r, w.rho_b).step(12).state()
    prm = oracle_params(p)
    e = state_errors(f, O.step(prm, O.init(prm, w.rho_r, w.rho_b), 12))
    assert e["worst"] <= TOL[storage], e

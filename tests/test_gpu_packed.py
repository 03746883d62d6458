"""The packed raw form (19 totals, phase, recolouring vector per site) that
one-read steps write, and the tile that decodes it: every row count at chunk and
tile remainders against the oracle, and a state that changes between the pair
arrays (set, imported, loaded) and the packed form.

Tolerances: FP64 1e-12 and FP32 1e-5 relative L2 against the oracle, as the
parity tests; equal bits where the same values are read through another form.
"""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2005_12764_amd import lb
from paper_2005_12764_amd import workloads as W
from tests.helpers import oracle_params, state_errors

pytestmark = pytest.mark.gpu

TOL = {W.F64: 1e-12, W.F32: 1e-5}
MOVING = ((0, 0.004, -0.002), (0, -0.003, 0.002), (0.005, 0, 0.001), (-0.004, 0, 0.003), (-0.01, 0.002, 0),
          (0.01, -0.001, 0))


def _case(n, bc, storage, moving):
    nx, ny, nz = n
    rr, rb, u = W.random_state(23, (nz, ny, nx))
    p = W.base_params(nx, ny, nz, bc=bc, storage=storage, tau_r=0.7, tau_b=1.2, A=0.01,
                      body_force=(1e-5, -2e-6, 3e-6))
    if moving:
        p["wall_velocity"] = MOVING
    return p, rr, rb, u


@pytest.mark.parametrize("rows,planes", [(4, 1), (4, 3), (8, 1), (8, 5), (16, 4), (0, 0)])
@pytest.mark.parametrize("n,bc,moving", [((65, 17, 7), (0, 0, 0), False), ((64, 9, 5), (0, 1, 1), False),
                                         ((66, 8, 6), (1, 1, 1), True), ((3, 33, 2), (1, 0, 0), False)],
                         ids=["x65", "walls_yz", "moving", "narrow_x"])
@pytest.mark.parametrize("storage", [W.F64, W.F32])
def test_tile_edges_against_the_oracle(storage, n, bc, moving, rows, planes):
    p, rr, rb, u = _case(n, bc, storage, moving)
    lb.lb_set_tiles(lb.TILES_ONE_READ, storage, rows, planes)
    try:
        with lb.Lattice(dict(p, kernel=lb.KERNEL_FUSED)) as L:
            L.init(rr, rb, u).step(9)
            f = L.state()
            m = L.moments()
            # saved as pair arrays, read back, and stepped on
            ck = L.save_raw()
            L.step(3)
            straight = L.state()
            L.load_raw(ck)
            assert np.array_equal(L.state(), f)
            L.step(3)
            assert np.array_equal(L.state(), straight)
    finally:
        lb.lb_set_tiles(lb.TILES_ONE_READ, storage, 0, 0)
    prm = oracle_params(p)
    ref = O.step(prm, O.init(prm, rr, rb, u), 9)
    e = state_errors(f, ref)
    assert e["worst"] <= TOL[storage], e
    for a, b in zip(m[:2], (ref[0].sum(0), ref[1].sum(0))):
        assert np.abs(a - b).max() <= TOL[storage]


def test_changing_the_tile_shape_between_steps():
    # the phase sums of a packed state are made again for other tile boxes
    p, rr, rb, u = _case((70, 20, 9), (0, 1, 0), W.F64, False)
    with lb.Lattice(dict(p, kernel=lb.KERNEL_FUSED)) as L:
        L.init(rr, rb, u).step(4)
        lb.lb_set_tiles(lb.TILES_ONE_READ, W.F64, 4, 2)
        try:
            L.step(4)
        finally:
            lb.lb_set_tiles(lb.TILES_ONE_READ, W.F64, 0, 0)
        L.step(4)
        f = L.state()
    prm = oracle_params(p)
    assert state_errors(f, O.step(prm, O.init(prm, rr, rb, u), 12))["worst"] <= 1e-12


@pytest.mark.parametrize("storage", [W.F64, W.F32])
def test_batched_job_without_steps_keeps_its_initial_state(storage):
    p, rr, rb, u = _case((40, 12, 6), (0, 0, 0), storage, False)
    with lb.Lattice(p) as L:
        L.init(rr, rb, u)
        want, moments = L.state(), L.moments()
    with lb.Batch(2, 1 << 26, storage, graph_steps=2) as B:
        a, b = B.add(p, rr, rb, u, steps=0), B.add(p, rr, rb, u, steps=3)
        B.step(4)
        assert np.array_equal(B.state(a), want)
        assert all(np.array_equal(g, r) for g, r in zip(B.moments(a), moments))
        assert B.job_steps(b) == 3

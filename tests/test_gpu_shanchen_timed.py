"""lb_step_timed of Shan-Chen lattices: the density pass of two-pass steps has its
own time, one-pass steps have none.

The density pass reads all 38 values of a site, the collide pass reads and writes
them: by bytes a third of the step.  Bound: a tenth, some 20 us here, where the
interval between two events with nothing between them takes under 10.
"""
import pytest

from paper_2005_12764_amd import lb
from paper_2005_12764_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage,shear,passes", [(W.F64, 0.0, 2), (W.F64, 0.01, 2), (W.F32, 0.01, 2), (W.F32, 0.0, 1)])
def test_pass_times(storage, shear, passes):
    n = 112
    rr, rb, u = W.random_state(47, (n, n, n))
    p = W.base_params(n, n, n, bc=(0, 0, 1), storage=storage)
    p.update(model=lb.MODEL_SHAN_CHEN, g_sc=0.2, A=0.0)
    if shear:
        p["wall_velocity"] = ((0, 0, 0),) * 4 + ((-shear, 0, 0), (shear, 0, 0))
    with lb.Lattice(p) as L:
        L.init(rr, rb, u).step(3)
        density, collide, step = lb.lb_step_timed(L.h, 5)
    assert (density > 0.1 * step) == (passes == 2), (density, collide, step)
    assert collide > 0.4 * step
    assert abs(density + collide - step) < 0.05 * step

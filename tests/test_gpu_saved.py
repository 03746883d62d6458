"""Saved raw states: equal states are equal bytes, whatever the buffers held before,
in host memory and in device memory of any alignment."""
import ctypes

import numpy as np
import pytest

from paper_2005_12764_amd import lb
from paper_2005_12764_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("steps", [0, 1, 4])
@pytest.mark.parametrize("storage", [W.F64, W.F32])
def test_equal_states_are_saved_as_equal_bytes(storage, steps):
    import torch
    nx, ny, nz = 33, 10, 7
    p = W.base_params(nx, ny, nz, bc=(0, 1, 0), storage=storage, tau_r=0.7, tau_b=1.2, A=0.01)
    fields, other = W.random_state(3, (nz, ny, nx)), W.random_state(4, (nz, ny, nx))
    with lb.Lattice(p) as L, lb.Lattice(p) as M:
        want = L.init(*fields).step(steps).save_raw()
        state = L.state()
        M.init(*other).step(4)
        M.load_raw(M.save_raw())
        M.step(3)
        M.init(*fields).step(steps)
        assert np.array_equal(M.state(), state)
        for offset in (0, 4, 8):
            d = torch.full((want.size + 64,), 7, dtype=torch.uint8, device="cuda")
            torch.cuda.synchronize()
            lb._check(lb.lib().lb_save_raw(M.h, ctypes.c_void_p(d.data_ptr() + offset), 1))
            torch.cuda.synchronize()
            got = d.cpu().numpy()
            assert np.array_equal(got[offset:offset + want.size], want)
            assert (got[:offset] == 7).all() and (got[offset + want.size:] == 7).all()
        assert np.array_equal(M.save_raw(), want)
        assert np.array_equal(M.step(2).state(), L.step(2).state())   # saving leaves the run unchanged
        M.load_raw(want)
        assert np.array_equal(M.step(2).state(), L.state())

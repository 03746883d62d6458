"""Lattices around the one-read step's 32-bit buffer offsets: 16-bit storage fits them
up to 113,025,000 sites (38 bytes each), pairs in FP32 only up to 107 million with
five arrays a resource.

Two ways of stepping agree as the parity tests' storage does (fp16 2e-4 of densities
of order one); the same kernels give equal bits.
"""
import ctypes

import pytest

from paper_2005_12764_amd import lb
from paper_2005_12764_amd import workloads as W

pytestmark = pytest.mark.gpu

CENTRES = [(60.0, 60.0, 60.0), (70.0, 240.0, 200.0), (300.0, 100.0, 350.0)]
RADII = [30.0, 40.0, 50.0]


def _fields(call, shape):
    import torch
    out = [torch.empty(shape, device="cuda") for _ in range(2)]
    torch.cuda.synchronize()
    call(*[ctypes.c_void_p(o.data_ptr()) for o in out])
    torch.cuda.synchronize()
    return out


def test_16_bit_job_near_the_limit_is_admitted():
    n = 478                                          # 109.2 million sites
    p = W.base_params(n, n, n, storage=W.F16, tau_r=0.8, tau_b=0.8, A=0.005)
    with lb.Lattice(p) as L:
        L.init_droplets(CENTRES, RADII).step(4)
        ref = _fields(lambda r, b: lb._check(lb.lib().lb_moments(L.h, r, b, None, lb.DTYPE_F32, 1, None)), (n, n, n))
    with lb.Batch(1, lb.lb_batch_job_bytes(p) + (1 << 20), W.F16, graph_steps=2) as B:
        slot = B.add_droplets(p, CENTRES, RADII, steps=4)
        B.step(4)
        got = _fields(lambda r, b: lb._check(lb.lib().lb_batch_moments(B.h, slot, r, b, None, lb.DTYPE_F32, 1, None)),
                      (n, n, n))
    for a, b in zip(got, ref):
        assert float((a - b).abs().max()) <= 2e-4
    assert float(ref[0].amax()) > 0.9 and float(ref[1].amax()) > 0.9


def test_moving_walls_beyond_the_limit_take_two_passes():
    n = 484                                          # 113.4 million sites
    p = W.base_params(n, n, n, bc=(0, 0, 1), storage=W.F16, tau_r=0.8, tau_b=0.8, A=0.005)
    p["wall_velocity"] = ((0, 0, 0),) * 4 + ((-0.01, 0, 0), (0.01, 0, 0))
    out = []
    for kernel in (lb.KERNEL_FUSED, lb.KERNEL_TWOPASS):
        with lb.Lattice(dict(p, kernel=kernel)) as L:
            L.init_droplets(CENTRES, RADII).step(3)
            out.append(_fields(lambda r, b: lb._check(lb.lib().lb_moments(L.h, r, b, None, lb.DTYPE_F32, 1, None)),
                               (n, n, n)))
    for a, b in zip(*out):
        assert bool((a == b).all())


def test_raw_moving_walls_beyond_the_limit_continue_a_saved_state():
    import torch
    n = 378                                          # 54.0 million sites, FP64
    p = W.base_params(n, n, n, bc=(0, 0, 1), storage=W.F64, tau_r=0.8, tau_b=0.8, A=0.005)
    p["wall_velocity"] = ((0, 0, 0),) * 4 + ((-0.01, 0, 0), (0.01, 0, 0))
    out = []
    with lb.Lattice(dict(p, kernel=lb.KERNEL_TWOPASS)) as L:
        L.init_droplets(CENTRES, RADII).step(1)
        image = torch.empty(L.state_bytes(), dtype=torch.uint8, device="cuda")
        torch.cuda.synchronize()
        lb._check(lb.lib().lb_save_raw(L.h, ctypes.c_void_p(image.data_ptr()), 1))
        L.step(2)
        out.append(_fields(lambda r, b: lb._check(lb.lib().lb_moments(L.h, r, b, None, lb.DTYPE_F32, 1, None)),
                           (n, n, n)))
    with lb.Lattice(dict(p, kernel=lb.KERNEL_FUSED)) as L:
        lb._check(lb.lib().lb_load_raw(L.h, ctypes.c_void_p(image.data_ptr()), 1))
        L.step(2)
        out.append(_fields(lambda r, b: lb._check(lb.lib().lb_moments(L.h, r, b, None, lb.DTYPE_F32, 1, None)),
                           (n, n, n)))
    for a, b in zip(*out):
        assert bool((a == b).all())

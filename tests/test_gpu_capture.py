"""Steps and readings captured into a graph on a lattice's own stream: every replay
acts on the state as an eager call does, whatever form that state has in memory.

Tolerances: FP64 1e-12 and FP32 1e-5 relative L2 against the oracle (the parity
tests'); equal bits where the same kernels run eagerly.
"""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2005_12764_amd import lb
from paper_2005_12764_amd import workloads as W
from tests.helpers import oracle_params, state_errors

pytestmark = pytest.mark.gpu

TOL = {W.F64: 1e-12, W.F32: 1e-5}
N = (70, 20, 9)
SHAPE = (9, 20, 70)


def _case(storage, seed=51, bc=(0, 1, 0)):
    nx, ny, nz = N
    rr, rb, u = W.random_state(seed, (nz, ny, nx))
    return W.base_params(nx, ny, nz, bc=bc, storage=storage, tau_r=0.7, tau_b=1.2, A=0.01), rr, rb, u


def _graph(stream, fn):
    import torch
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=stream, capture_error_mode="thread_local"):
        fn()
    return g


def _replay(g, stream, n=1):
    import torch
    with torch.cuda.stream(stream):
        for _ in range(n):
            g.replay()
            torch.zeros(1000, device="cuda").add_(1)   # eager work between replays
    torch.cuda.synchronize()


@pytest.mark.parametrize("storage", [W.F64, W.F32])
def test_steps_captured_on_a_state_just_set(storage):
    import torch
    p, rr, rb, u = _case(storage)
    prm = oracle_params(p)
    ref = O.init(prm, rr, rb, u)
    s = torch.cuda.Stream()
    with lb.Lattice(p, stream=s) as L:
        L.init(rr, rb, u)
        g = _graph(s, lambda: L.step(2))
        for n in (1, 2):
            _replay(g, s, n)
            ref = O.step(prm, ref, 2 * n)
            assert state_errors(L.state(), ref)["worst"] <= TOL[storage]
        L.step(2)                                   # eager steps between replays
        _replay(g, s)
        ref = O.step(prm, ref, 4)
        assert state_errors(L.state(), ref)["worst"] <= TOL[storage]
        L.set_state(ref)                            # and a state set between them
        _replay(g, s)
        assert state_errors(L.state(), O.step(prm, ref, 2))["worst"] <= TOL[storage]


@pytest.mark.parametrize("storage", [W.F64, W.F32])
def test_readings_captured_on_a_state_just_set(storage):
    import torch
    p, rr, rb, u = _case(storage)
    real = torch.float64 if storage == W.F64 else torch.float32
    out = torch.empty((2, 19) + SHAPE, dtype=real, device="cuda")
    mom = [torch.empty(k + SHAPE, dtype=real, device="cuda") for k in ((), (), (3,))]
    torch.cuda.synchronize()
    s = torch.cuda.Stream()
    with lb.Lattice(p, stream=s) as L:
        L.init(rr, rb, u)

        def read():
            lb.lb_get_state(L.h, out)
            lb.lb_moments(L.h, *mom)
        g = _graph(s, read)
        for n in (0, 2):
            L.step(n)
            _replay(g, s)
            want, m = L.state(), L.moments()
            eps = 1e-15 if storage == W.F64 else 6e-8   # the outputs' rounding of values below 1
            assert np.abs(out.cpu().numpy() - want).max() <= eps
            assert all(np.abs(a.cpu().numpy() - b).max() <= 2 * eps for a, b in zip(mom, m))


@pytest.mark.parametrize("storage", [W.F64, W.F32, W.F16, W.BF16])
def test_steps_captured_on_a_stepped_state_keep_the_one_read_step(storage):
    import torch
    p, rr, rb, u = _case(storage)
    s = torch.cuda.Stream()
    with lb.Lattice(p, stream=s) as L, lb.Lattice(p) as E:
        L.init(rr, rb, u).step(3)
        E.init(rr, rb, u).step(3)
        g = _graph(s, lambda: L.step(2))
        assert L.kernel == lb.KERNEL_FUSED
        for n in (1, 3):
            _replay(g, s, n)
            assert np.array_equal(L.state(), E.step(2 * n).state())


@pytest.mark.parametrize("storage", [W.F64, W.F32, W.F16, W.BF16])
def test_a_restart_captured_whole(storage):
    import torch
    p, rr, rb, u = _case(storage)
    real = torch.float64 if storage == W.F64 else torch.float32
    states = []
    for seed in (1, 2, 3):
        with lb.Lattice(p) as E:
            states.append(E.init(*_case(storage, seed)[1:]).state().astype(np.float64 if storage == W.F64 else np.float32))
    f, out = (torch.empty((2, 19) + SHAPE, dtype=real, device="cuda") for _ in range(2))
    torch.cuda.synchronize()
    s = torch.cuda.Stream()
    with lb.Lattice(p, stream=s) as L, lb.Lattice(p) as E:
        for k in range(2):                          # (a 16-bit lattice then holds the buffer of set states)
            L.set_state(states[k])
            L.step(1)

        def restart():
            lb.lb_set_state(L.h, f)
            L.step(3)
            lb.lb_get_state(L.h, out)
        g = _graph(s, restart)
        assert L.kernel == lb.KERNEL_FUSED
        for st in (states[2], states[0], states[1]):
            f.copy_(torch.from_numpy(st))
            torch.cuda.synchronize()
            _replay(g, s)
            E.set_state(st)
            assert np.array_equal(out.cpu().numpy(), E.step(3).state(dtype=st.dtype))


@pytest.mark.parametrize("storage", [W.F16, W.BF16])
def test_first_step_of_16_bits_is_not_captured_alone(storage):
    import torch
    p, rr, rb, u = _case(storage)
    s = torch.cuda.Stream()
    with lb.Lattice(p, stream=s) as L, lb.Lattice(p) as E:
        x = torch.zeros(8, device="cuda")
        for k in range(2):
            L.init(rr, rb, u)
            torch.cuda.synchronize()

            def steps():
                x.add_(1)
                with pytest.raises(lb.LbError) as e:
                    L.step(2)
                assert e.value.code == lb.LB_ESTATE
            _graph(s, steps)
            assert np.array_equal(L.step(2).state(), E.init(rr, rb, u).step(2).state())

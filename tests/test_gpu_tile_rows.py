"""Twelve rows asked for through lb_set_tiles are the rows taken, and the tuner finds
shapes of the one-read step in 16-bit storage."""
import numpy as np
import pytest

from paper_2005_12764_amd import autotune as T
from paper_2005_12764_amd import lb
from paper_2005_12764_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage", [W.F16, W.BF16])
def test_rows_asked_for_are_taken(storage, monkeypatch):
    w = W.two_droplets(n=(70, 29, 19), R=6, gap=2.0, A=0.01, nc_strength=0.03, nc_range=2)
    p = dict(w.params, storage=storage, kernel=lb.KERNEL_FUSED)

    def run():
        with lb.Lattice(p) as L:
            return L.init(w.rho_r, w.rho_b).step(12).state()
    monkeypatch.setenv("LB_SINGLE_TY", "12")
    monkeypatch.setenv("LB_TZ", "5")
    want = run()
    monkeypatch.delenv("LB_SINGLE_TY")
    other = run()
    monkeypatch.delenv("LB_TZ")
    lb.lb_set_tiles(lb.TILES_ONE_READ, storage, 12, 5)
    try:
        assert np.array_equal(run(), want)
        assert not np.array_equal(other, want)       # (the tile boxes move the rounding)
    finally:
        lb.lb_set_tiles(lb.TILES_ONE_READ, storage, 0, 0)


def test_tuner_times_the_one_read_step_in_16_bits():
    arch = T.device_arch()
    cache = {}
    out = T.tune_lattice(32, W.F16, arch, cache, steps=4, log=lambda m: print(m, flush=True))
    e = out[T.cache_key(arch, W.F16, lb.TILES_ONE_READ, "small")]
    assert {r["ty"] for r in e["timings"] if r["ms"] is not None} >= {4, 8, 12}

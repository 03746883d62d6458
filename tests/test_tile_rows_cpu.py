"""Twelve rows of the one-read step, its own choice in 16-bit storage, can be asked for
there and nowhere else, and the tuner times them (no GPU)."""
import pytest

from paper_2005_12764_amd import autotune as T
from paper_2005_12764_amd import lb
from paper_2005_12764_amd import workloads as W


@pytest.mark.parametrize("kind", [lb.TILES_PHASE, lb.TILES_COLLIDE, lb.TILES_ONE_READ, lb.TILES_BATCH])
@pytest.mark.parametrize("storage", [W.F64, W.F32, W.F16, W.BF16])
def test_twelve_rows(kind, storage):
    if kind == lb.TILES_ONE_READ and storage in (W.F16, W.BF16):
        lb.lb_set_tiles(kind, storage, 12, 0)
        lb.lb_set_tiles(kind, storage, 0, 0)
        assert (12, 0) in T.candidates(kind, storage)
    else:
        with pytest.raises(lb.LbError):
            lb.lb_set_tiles(kind, storage, 12, 0)
        assert T.candidates(kind, storage) == T.CANDIDATES[kind]

"""Edges of the kernels' tiles, remainders and dispatch rules, against numpy or the oracle."""
import numpy as np
import pytest
import torch

from gpu_common import dev, lib, note

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n, n_tiles", [(1, 1), (2047, 64), (2049, 1), (70_001, 4096), (70_001, 4097), (40_000, 12_000)])
@pytest.mark.parametrize("kind", ["mixed", "equal"])
def test_tile_max_at_block_and_table_edges(n, n_tiles, kind):
    """One batch more or less than a block takes, tables of 4096 tiles in LDS and of 4097 in memory, more tiles than
    a block has templates; values with infinities and ties, or all equal (every template attains its maximum)."""
    tfsc = lib()
    rng = np.random.default_rng(n + n_tiles)
    note(f"tile max: {n} values, {n_tiles} tiles, {kind}")
    stat = np.zeros(n) if kind == "equal" else np.round(rng.exponential(30.0, n), 1)
    if kind == "mixed" and n > 8:
        stat[rng.integers(0, n, 4)] = np.inf
        stat[rng.integers(0, n, 4)] = np.nan
    tile = rng.integers(-1, n_tiles, n).astype(np.int32)
    mx, arg = (t.cpu().numpy() for t in tfsc.tile_max(dev(stat), dev(tile), n_tiles))
    ok = (tile >= 0) & (stat >= 0.0)
    rmx = np.zeros(n_tiles)
    np.maximum.at(rmx, tile[ok], stat[ok])
    rarg = np.full(n_tiles, n, np.int64)
    at = np.flatnonzero(ok & (stat == rmx[np.maximum(tile, 0)]))
    np.minimum.at(rarg, tile[at], at)
    rarg[rarg == n] = -1
    assert np.array_equal(mx, rmx) and np.array_equal(arg, rarg)

"""GPU parity of candidate clustering where the components meet the edges of
the 1024-position tiles that are linked on their own first (exact)."""
import numpy as np
import pytest

from oracle import CAND_DTYPE
from test_gpu_cluster import _random_cands, check

pytestmark = pytest.mark.gpu


def _cands(sample, dm, width, snr):
    c = np.empty(len(sample), dtype=CAND_DTYPE)
    c["sample"], c["dm_idx"], c["width"], c["snr"] = sample, dm, width, snr
    return c


@pytest.mark.parametrize("n", [1023, 1024, 1025, 2047, 2048, 2049, 5000])
def test_tile_edges(n):
    rng = np.random.default_rng(n)
    # one chain through every tile, its steps at the tolerance; then with every 700th link missing
    t = np.arange(n) * 8
    snr = rng.permutation(n).astype(np.float32) + 6
    order = rng.permutation(n)
    check(_cands(t, np.full(n, 3), np.full(n, 4), snr)[order], 8, 0, 0, "chain")
    t = t + np.arange(n) // 700
    check(_cands(t, np.full(n, 3), np.full(n, 4), snr)[order], 8, 0, 0, "broken-chain")
    # one sample, so one time row: cells of a few trials, and one cell for all
    d = rng.permutation(4 * n)[:n]
    check(_cands(np.full(n, 77), d, np.full(n, 1), snr), 5, 3, 1, "one-row")
    check(_cands(np.full(n, 77), d, np.full(n, 1), snr), 5, 4 * n, 1, "one-cell")
    # equal S/N: the tie-break decides between members of different tiles
    c = _random_cands(rng, n, 0, 4 * n, 6, 5, ties=True)
    c["snr"] = 7.0
    check(c, 30, 2, 4, "ties")


def test_time_rows_longer_than_a_tile():
    # rows of cells that hold 3000 candidates each: the compared positions lie up to three tiles ahead
    rng = np.random.default_rng(3)
    s = np.repeat(np.arange(4) * 10, 3000)
    d = np.concatenate([np.sort(rng.permutation(20000)[:3000]) for _ in range(4)])
    c = _cands(s, d, 1 << rng.integers(0, 3, size=s.size), rng.uniform(6, 30, size=s.size).astype(np.float32))
    check(c[rng.permutation(c.size)], 10, 4, 1, "long-rows")
    check(c[rng.permutation(c.size)], 9, 2, 0, "long-rows-apart")


@pytest.mark.parametrize("n", [1, 2047, 2048, 2049, 6145])
def test_cell_counts(n):
    # workgroups count 2048 candidates in a table of their own: every one in a
    # cell of its own (the table as full as it gets), a few cells each, one cell
    rng = np.random.default_rng(n)
    snr = rng.permutation(n).astype(np.float32) + 6
    one = np.full(n, 4)
    check(_cands(rng.permutation(n) * 1000, np.full(n, 3), one, snr), 2, 0, 0, "own-cells")
    check(_cands(rng.integers(0, 7, size=n) * 1000, rng.integers(0, 3, size=n) * 50, one, snr), 2, 1, 0, "few-cells")
    check(_cands(np.full(n, 9), np.full(n, 3), one, snr), 2, 0, 0, "one-cell")

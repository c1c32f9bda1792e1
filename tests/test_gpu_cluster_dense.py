"""GPU parity of candidate clustering in few and in many cells: tolerances that
put a set into few cells, where nearly every pair is compared, most reach past
the positions held in LDS and several workgroups share a tile's positions; and
ranges that take all the cells there are (exact)."""
import numpy as np
import pytest

from test_gpu_cluster import check
from test_gpu_cluster_tiles import _cands

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1025, 3073, 4097, 9000])
def test_one_cell(n):
    rng = np.random.default_rng(n)
    snr = rng.permutation(n).astype(np.float32) + 6
    w = 1 << rng.integers(0, 12, size=n)
    # all linked; linked by width alone, so in twelve components; by trial alone, so few
    check(_cands(rng.integers(0, 1000, size=n), rng.integers(0, 50, size=n), w, snr), 2000, 100, 12, "all-linked")
    check(_cands(rng.integers(0, 1000, size=n), rng.integers(0, 50, size=n), w, snr), 2000, 100, 0, "by-width")
    check(_cands(rng.integers(0, 1000, size=n), rng.permutation(2 * n)[:n], np.ones(n, int), snr), 2000, 1, 0, "by-trial")


def test_wide_tolerances():
    # rows of some thousand candidates: joins within LDS, past it and into the tile after next
    n = 12000
    rng = np.random.default_rng(5)
    snr = rng.permutation(n).astype(np.float32) + 6
    s, d = rng.integers(0, 1 << 20, size=n), rng.integers(0, 1000, size=n)
    check(_cands(s, d, 1 << rng.integers(0, 12, size=n), snr), 200000, 10, 1, "wide")
    check(_cands(s, d, 1 << rng.integers(0, 12, size=n), snr), 100, 1000, 0, "tall")


@pytest.mark.parametrize("span,trials", [(1 << 30, 4), (1 << 16, 1 << 20), (3 << 18, 6), (1 << 22, 1)])
def test_every_cell(span, trials):
    n = 3000
    rng = np.random.default_rng(span % 1000 + trials)
    s = np.concatenate([rng.integers(0, span, size=n), [0, span - 1]])
    s[1:n:2] = s[0:n - 1:2] + rng.integers(0, 3, size=n // 2)  # half of them near another
    d = np.concatenate([rng.integers(0, trials, size=n), [0, trials - 1]])
    d[1:n:2] = d[0:n - 1:2]
    check(_cands(s, d, np.full(n + 2, 2), rng.permutation(n + 2).astype(np.float32) + 6), 1, 0, 0, "every-cell")

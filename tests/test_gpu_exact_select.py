"""GPU parity of the block statistics of data too spread for any histogram, which
every block selects from its window: windows about the eight wave loads taken
at a time, digits shared by all lanes, by some, by none. Exact."""
import numpy as np
import pytest

import oracle
from test_gpu_parity import gpu_search

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L", [1, 2, 50, 64, 65, 130, 511, 512, 513, 576, 1000, 1024, 4096, 9001])
@pytest.mark.parametrize("bins", [4096, 16384])
def test_window_lengths(L, bins):
    n = 5000
    rng = np.random.default_rng(L)
    x = np.stack([
        200000.0 + np.round(rng.normal(0.0, 60000.0, size=n)),                  # upper digits shared
        np.round(rng.uniform(-8000000.0, 8000000.0, size=n)),                   # every digit spread, both signs
        np.where(rng.random(n) < 0.5, -70000.0, 65536.0 * rng.integers(-3, 4, size=n)),  # few values far apart
        np.where((np.arange(n) // 700) % 2, 5.0, np.round(rng.normal(0.0, 90000.0, size=n))),  # in and out of the select
    ]).astype(np.float32)
    print("exact select", L, bins, flush=True)
    got, med, mad = gpu_search(x, 8, L, 5.0, hist_bins=bins, capacity=8 * x.size)
    ref, rm, rd = oracle.search(x, 8, L, 5.0, with_stats=True)
    assert np.array_equal(med, rm) and np.array_equal(mad, rd)

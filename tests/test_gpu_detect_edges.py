"""GPU parity of the detection where a wave's window ends are all valid, partly
valid or not at all: rows about multiples of a step, segments of one step up to
the whole row, runs that stay open across quiet and full stretches."""
import numpy as np
import pytest

import oracle
from parity import exact_equal
from test_gpu_parity import gpu_search

pytestmark = pytest.mark.gpu


def rows(n, rng):
    x = 32768.0 + np.round(rng.normal(0.0, 1024.0, size=(5, n)))
    x[0, : n // 2] += 400.0                                   # wide windows above, narrow ones quiet
    x[1, max(0, n - 1100):] += 9000.0                          # a run into the row's end
    x[2, :700] += 9000.0                                       # a run from its start
    for at in range(1000, n, 1024):                            # runs over the steps' edges
        x[3, at:at + 50] += 20000.0
    x[4, n // 3:n // 3 + 2600] += 30000.0                      # full groups over several steps
    return x.astype(np.float32)


@pytest.mark.parametrize("top", [1, 8, 64, 1024, 4096])
@pytest.mark.parametrize("n", [1, 63, 1024, 4097, 9215, 16385])
def test_validity_edges(n, top):
    if top > n:
        pytest.skip("a row holds its widest window")
    x = rows(n, np.random.default_rng(n + top))
    L = min(n, 3000)
    ref = oracle.search(x, top, L, 5.0)
    for seg in (0, 1024, 2048, 8192):                          # one to seventeen segments a row, eight and nine
        print("detect edges", n, top, seg, flush=True)
        got, _, _ = gpu_search(x, top, L, 5.0, detect_seg=seg, capacity=4 * ref.size + 64)
        assert exact_equal(got, ref), (n, top, seg)


@pytest.mark.parametrize("every", [2, 11, 40, 700, 5000])
def test_staged_candidates(every):
    # from several hundred candidates a step (past the staging buffers) to none for several steps
    n, top, L = 30000, 16, 3000
    x = 32768.0 + np.round(np.random.default_rng(every).normal(0.0, 1024.0, size=(3, n)))
    x[0, ::every] += 30000.0
    x[1, : n // 2 : every] += 30000.0
    x[2, n - 1200 :: every] += 30000.0
    x = x.astype(np.float32)
    ref = oracle.search(x, top, L, 6.0)
    for seg in (0, 1024, 8192):
        print("staged candidates", every, seg, ref.size, flush=True)
        got, _, _ = gpu_search(x, top, L, 6.0, detect_seg=seg, capacity=ref.size)
        assert exact_equal(got, ref), (every, seg)

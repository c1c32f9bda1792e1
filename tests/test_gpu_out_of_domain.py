"""Rows outside the input domain (saturating, infinite or undefined samples) have
unspecified results, but the launch ends and the other rows are untouched."""
import numpy as np
import pytest

import oracle
from test_gpu_parity import gpu_search

pytestmark = pytest.mark.gpu


def rows(kind, n, rng):
    x = 4000000.0 + np.round(rng.normal(0.0, 300.0, size=(8, n)))
    if kind == "saturated":    # a head at the lowest integer, spread by about its distance from the rest
        step = 128.0 * 782
        for r in range(8):
            head = 600 + 100 * r
            x[r, :head] = -2147483648.0 + step * rng.permutation(64).repeat(-(-head // 64))[:head]
    elif kind == "infinite":
        x[::2, : n // 3] = -np.inf
        x[1::2, n // 2:] = np.inf
    elif kind == "undefined":
        x[:, ::3] = np.nan
    elif kind == "huge":
        x *= np.round(10.0 ** rng.uniform(0.0, 30.0, size=(8, n)))
    return x


@pytest.mark.parametrize("seg", [0, 8, 64])
@pytest.mark.parametrize("kind", ["saturated", "infinite", "undefined", "huge"])
def test_other_rows_are_untouched(kind, seg):
    n, top, L = 20000, 64, 4096
    rng = np.random.default_rng(seg)
    x = np.concatenate([32768.0 + np.round(rng.normal(0.0, 1024.0, size=(1, n))), rows(kind, n, rng),
                        32768.0 + np.round(rng.normal(0.0, 1024.0, size=(1, n)))]).astype(np.float32)
    x[[0, -1], 700:740] += 9000.0
    print("out of domain", kind, seg, flush=True)
    got, med, mad = gpu_search(x, top, L, 5.0, stats_seg=seg, capacity=2 * x.size)
    ref, rm, rd = oracle.search(x[[0, -1]], top, L, 5.0, with_stats=True)
    assert np.array_equal(med[[0, -1]], rm) and np.array_equal(mad[[0, -1]], rd)
    got = got[(got["dm_idx"] == 0) | (got["dm_idx"] == 9)]
    got["dm_idx"] //= 9
    assert got.size == ref.size
    for f in ("sample", "dm_idx", "width", "snr"):
        assert np.array_equal(got[f], ref[f]), f

"""GPU parity of the per-width scales on series of few values, where the sampled
estimate lies a value or two off the median and the MAD is smaller than that.
Bit-exact against the oracle."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def check(x, top, L, what):
    import torch
    from paper_2512_00398_amd import sps
    print("width small values", what, x.shape, top, L, flush=True)
    with sps.Plan(x.shape[0], x.shape[1], top, L, 6.0) as p:
        c, m = p.width_stats(torch.from_numpy(x).cuda())
        torch.cuda.synchronize()
        c, m = c.cpu().numpy(), m.cpu().numpy()
    for r in range(x.shape[0]):
        rc, rm = oracle.width_stats(x[r], top, L)
        assert np.array_equal(c[r], rc), (what, r, c[r], rc)
        assert np.array_equal(m[r], rm), (what, r, m[r], rm)


@pytest.mark.parametrize("off", [-3, -2, -1, 1, 2, 3])
@pytest.mark.parametrize("n", [32768, 40000, 131136])
def test_estimate_beside_the_median(n, off):
    # Each 64 samples hold the same values (so every block's median is 0): 18 of
    # the median, 31 below it and 15 above. The sampled positions (3 mod 4) hold
    # 9 of `off` and 7 of the others, so the sampled median is `off` values away;
    # the MAD is 1 on one side and |off| on the other.
    if off < 0:
        values = np.r_[np.full(31, off), np.full(18, 0), np.full(15, 4)]
    else:
        values = np.r_[np.full(15, -4), np.full(18, 0), np.full(31, off)]
    sampled = np.r_[values[values == off][:9], values[values == 0][:4], values[abs(values) == 4][:3]]
    rest = list(values)
    for v in sampled:
        rest.remove(v)
    block = np.empty(64)
    block[3::4] = sampled
    block[np.arange(64) % 4 != 3] = rest
    x = 32768.0 + np.tile(block, (2, -(-n // 64)))[:, :n]
    x[1] = 65536.0 - x[1]
    check(x.astype(np.float32), 8, 640, ("beside", off))


@pytest.mark.parametrize("kind", ["few", "outlier", "bits", "sparse"])
@pytest.mark.parametrize("n", [43, 345, 5000, 32767, 46171])
def test_few_values(n, kind):
    rng = np.random.default_rng(n + len(kind))
    rows = 24
    if kind == "few":           # two to six values in uneven shares
        x = np.stack([rng.choice(rng.integers(-9, 10, size=6), p=rng.dirichlet(np.ones(6)), size=n) for _ in range(rows)])
    elif kind == "outlier":     # the sample's histogram has wide bins
        x = rng.integers(0, 4, size=(rows, n))
        for r in range(rows):
            x[r, rng.integers(0, n, size=3)] = rng.integers(-90000, 90000)
    elif kind == "bits":
        x = rng.integers(0, 2, size=(rows, n)) + rng.integers(0, 2, size=(rows, n)) * 2
    else:                       # mostly zeros
        x = np.where(rng.random((rows, n)) < 0.3, rng.integers(1, 4, size=(rows, n)), 0)
    check(x.astype(np.float32), min(64, 1 << int(np.log2(n))), min(n, 900), kind)


@pytest.mark.parametrize("kind", ["constant", "sampled-constant", "blanked", "padded", "two-runs", "rare"])
@pytest.mark.parametrize("n", [100, 5001, 32767, 33000, 131072 + 70])
def test_one_value_holds_much_of_the_series(n, kind):
    rng = np.random.default_rng(n + len(kind))
    x = np.full((6, n), 1000.0)
    noise = np.round(rng.normal(0.0, 200.0, size=(6, n)))
    if kind == "sampled-constant":  # every sampled position alike, the others not
        x += np.where(np.arange(n) % 4 == 3, 0.0, noise)
    elif kind == "blanked":         # rows blanked here and there, from nearly all to a tenth
        for r in range(6):
            x[r] += np.where(rng.random(n // 50 + 1).repeat(50)[:n] < 0.97 - 0.17 * r, 0.0, noise[r])
    elif kind == "padded":          # noise, then nothing; the last row all of it
        for r in range(6):
            x[r, : n * r // 5] += noise[r, : n * r // 5]
    elif kind == "two-runs":        # two values in long runs, from even to one in ten
        for r in range(6):
            x[r] += 3.0 * (rng.random(n // 100 + 1).repeat(100)[:n] < 0.5 - 0.08 * r)
    elif kind == "rare":
        x += np.where(rng.random((6, n)) < 0.02, 3.0, 0.0)
    check(x.astype(np.float32), min(4096, 1 << int(np.log2(n))), min(n, 700), kind)

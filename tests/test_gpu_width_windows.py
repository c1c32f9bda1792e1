"""GPU parity of the per-width scales where the sampled estimate and the exact
windows could go wrong: row lengths about the sampling thresholds, data that
its sample describes well, badly or not at all. Bit-exact against the oracle."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def rows(kind, n, rng):
    t = np.arange(n)
    x = 32768.0 + np.round(rng.normal(0.0, 1024.0, size=(2, n)))
    if kind == "pulses":        # ranges far wider than the scale
        for k in range(8):
            x[:, int(rng.integers(0, n - 1100)):][:, :1 << k] += 400000.0 / (1 << k)
    elif kind == "drift":       # wide boxcars follow the drift
        x += np.round(2048.0 * np.sin(2 * np.pi * t / 8192))
    elif kind == "every4th":    # the sampled positions are unlike the others
        x[:, ::4] += 30000.0
    elif kind == "levels":      # two values: windows with empty bins and with everything
        x = 32768.0 + 5000.0 * (rng.random((2, n)) < 0.5)
    elif kind == "flat":        # every series constant but for a few samples
        x = np.full((2, n), 32768.0)
        x[:, n // 2:n // 2 + 3] += 7.0
    elif kind == "rare":        # one row far noisier in its last tenth
        x[1, n - n // 10:] += np.round(rng.normal(0.0, 300000.0, size=n // 10))
    return x.astype(np.float32)


@pytest.mark.parametrize("kind", ["noise", "pulses", "drift", "every4th", "levels", "flat", "rare"])
@pytest.mark.parametrize("n,top,L", [(4096, 4096, 1000), (32767, 4096, 4096), (32768, 4096, 4096), (32771, 128, 900),
                                     (131071, 64, 4096), (131072, 4096, 9000), (140001, 1024, 3000)])
def test_width_statistics(kind, n, top, L):
    import torch
    from paper_2512_00398_amd import sps
    rng = np.random.default_rng(n + len(kind))
    x = rows(kind, n, rng)
    print("width windows", kind, n, top, L, flush=True)
    with sps.Plan(2, n, top, L, 6.0) as p:
        c, m = p.width_stats(torch.from_numpy(x).cuda())
        torch.cuda.synchronize()
        c, m = c.cpu().numpy(), m.cpu().numpy()
    for r in range(2):
        rc, rm = oracle.width_stats(x[r], top, L)
        assert np.array_equal(c[r], rc), (kind, n, r)
        assert np.array_equal(m[r], rm), (kind, n, r)

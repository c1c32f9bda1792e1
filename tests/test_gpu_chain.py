"""GPU parity of the block statistics where the baseline moves fast: the walk
from block to block, recentring, refilling and the exact select, and the edges
of the interior blocks. Medians and MADs bit-exact against the oracle."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def sps():
    from paper_2512_00398_amd import sps as m
    return m


def rows(kind, ndm, n, rng):
    t = np.arange(n)
    noise = np.round(rng.normal(0.0, 1024.0, size=(ndm, n)))
    base = {"flood": 2048.0 * np.sin(2 * np.pi * t / 8192),     # walks of tens of bins a block
            "ramp": 8.0 * t,                                    # 512 a block: leaves the narrow windows, recentres
            "steep": 100.0 * t,                                 # 6400 a block: leaves the histogram at once
            "steps": 9000.0 * ((t // 700) % 2),                 # two levels: MADs too wide for the histogram
            "flat": 0.0 * t}[kind]
    x = noise + np.round(base) + 32768
    if kind == "flat":
        x = 32768 + np.round(noise / 2000)                       # few values, many ties
    x[:, n // 3] += 200000.0                                     # far outside the histogram
    return x.astype(np.float32)


@pytest.mark.parametrize("bins", [4096, 16384])
@pytest.mark.parametrize("kind", ["flood", "ramp", "steep", "steps", "flat"])
def test_moving_baseline(kind, bins):
    import torch
    m = sps()
    rng = np.random.default_rng(len(kind))
    # rows of 1 .. a few more blocks than the window, ragged ends, and chains
    # whose interior runs hold 0 to 9 blocks
    for n, L, seg in [(63, 64, 0), (1000, 4096, 0), (4096, 4096, 0), (4096 + 64 * 3, 4096, 0), (4096 + 64 * 9 + 1, 4096, 7),
                      (6000, 1000, 5), (6000, 65, 0), (9000, 3001, 11), (20000, 4096, 0)]:
        x = rows(kind, 3, n, rng)
        xd = torch.from_numpy(x).cuda()
        for window in (0, 1):
            print("chain case", kind, bins, n, L, seg, window, flush=True)
            with m.Plan(3, n, 4, L, 6.0) as p:
                p.set(m.ATTR_HIST_BINS, bins)
                p.set(m.ATTR_WINDOW, window)
                p.set(m.ATTR_STATS_SEG, seg)
                med, mad = p.block_stats(xd)
                torch.cuda.synchronize()
            _, rm, rd = oracle.search(x, 4, L, 6.0, with_stats=True, centered=bool(window))
            assert np.array_equal(med.cpu().numpy(), rm), (kind, n, L, seg, window)
            assert np.array_equal(mad.cpu().numpy(), rd), (kind, n, L, seg, window)


@pytest.mark.parametrize("kind", ["flood", "ramp", "steps"])
def test_moving_baseline_in_streams(kind):
    # windows that reach into the history, one gulp at a time and two streams in one push
    import torch
    from parity import exact_equal
    m = sps()
    rng = np.random.default_rng(17)
    gulp, L = 2048, 3000
    xs = [rows(kind, 2, 4 * gulp, rng), rows(kind, 3, 4 * gulp, rng)]
    plans = [m.Plan(x.shape[0], gulp, 16, L, 5.0) for x in xs]
    for p in plans:
        p.set(m.ATTR_MAX_CANDS, 1 << 15)
    for batched in (False, True):
        streams = [m.Stream(p) for p in plans]
        bufs = [p.alloc_cands() for p in plans]
        got = [[], []]

        def keep(i, off):
            c = m.cands_to_numpy(*bufs[i], plans[i].max_cands)
            a = np.empty(c.size, dtype=oracle.CAND_DTYPE)
            a["sample"] = c["sample"].astype(np.int64) + off
            a["dm_idx"], a["width"], a["snr"] = c["dm_idx"], c["width"], c["snr"]
            got[i].append(a)

        with m.Batch() as b:
            for k in range(4):
                gs = [torch.from_numpy(np.ascontiguousarray(x[:, k * gulp:(k + 1) * gulp])).cuda() for x in xs]
                print("chain stream case", kind, batched, k, flush=True)
                if batched:
                    offs = b.push(streams, gs, [c for c, _ in bufs], [n for _, n in bufs])
                else:
                    offs = [s.push(g, *buf) for s, g, buf in zip(streams, gs, bufs)]
                torch.cuda.synchronize()
                for i, off in enumerate(offs):
                    keep(i, off)
        for i, s in enumerate(streams):
            end = s.flush(*bufs[i])
            torch.cuda.synchronize()
            keep(i, end)
            s.close()
            ref = oracle.search(xs[i], 16, L, 5.0)
            assert exact_equal(oracle.sort_cands(np.concatenate(got[i])), ref), (kind, batched, i)
    for p in plans:
        p.close()

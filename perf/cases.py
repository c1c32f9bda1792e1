"""The work measured on this framework: searches, streams, batches, dedispersion,
RFI excision, clustering and the whole pipeline, through the public binding.

Sizes follow the workloads of the synthetic generator and the benchmark (64 x
16384 small blocks, 1024 x 2^20 large ones, thousands of rows per streamed
gulp, files and beams of uneven shapes, 1024-channel filterbanks dedispersed
to 1024 trials in 2^18-sample chunks) and the ragged ones of the tests. Inputs
are drawn on the GPU from the seed: integer Gaussian noise of the generator's
mean and sigma with its sinusoidal drift (period 8192, which a 16384-sample
median does not follow and which floods the search with runs, or a slow one
that the baseline removes) and boxcar pulses on neighbouring rows; filterbanks
are 8-bit noise with dispersed pulses, broadband bursts and noisy channels.

Candidates come from the library in no fixed order, so a pass ends as a
program that reads them does: sorted by (row, width, sample).
"""
import math

import torch

from paper_2512_00398_amd import sps

MU, SIGMA, THRESH = 32768.0, 1024.0, 6.0
F_LO_MHZ, F_HI_MHZ = 1050.0, 1450.0
INVALID = (1 << 63) - 1
CLUSTER_TOL = (32, 3, 2)  # samples, trials, log2 widths: the benchmark's
MASK_K, ZERO_OFFSET = 4, 64
FLOOD, SLOW = 8192, 1 << 20  # drift periods in samples
UNSORTED = 1 << 16  # candidate buffers up to this many records are sorted whole


def listed():
    return [
        # many small blocks one after another: launches and short rows dominate
        {"name": "search_small", "kind": "search", "blocks": 8, "ndm": 64, "nsamp": 16384, "max_width": 64,
         "baseline": 4096, "drift": FLOOD, "window": 0, "norm": 0},
        # the benchmark's block: 67 s at 64 us and 1024 trials, with its drift
        {"name": "search_block", "kind": "search", "blocks": 1, "ndm": 1024, "nsamp": 1 << 20, "max_width": 4096,
         "baseline": 16384, "drift": FLOOD, "window": 0, "norm": 0},
        # a ragged block, windows centred, one noise scale per row
        {"name": "search_ragged", "kind": "search", "blocks": 1, "ndm": 333, "nsamp": 100003, "max_width": 512,
         "baseline": 5001, "drift": SLOW, "window": 1, "norm": 1},
        # one noise scale per filtered series
        {"name": "search_width_scale", "kind": "search", "blocks": 1, "ndm": 256, "nsamp": 131072,
         "max_width": 4096, "baseline": 4096, "drift": SLOW, "window": 0, "norm": 2},
        # a long observation gulp by gulp from two input buffers, captured graphs
        {"name": "stream_gulps", "kind": "stream", "ndm": 2048, "nsamp": 1 << 16, "gulps": 2, "max_width": 4096,
         "baseline": 16384, "drift": FLOOD, "norm": 0},
        # a serving step: one gulp of each of several beams in one launch
        {"name": "serve_beams", "kind": "serve", "beams": 4, "ndm": 700, "nsamp": 1 << 16, "max_width": 4096,
         "baseline": 16384, "drift": FLOOD},
        # files of uneven shapes in one launch
        {"name": "batch_files", "kind": "batch", "files": 10, "ndm": 256, "nsamp": 1 << 17, "max_width": 4096,
         "baseline": 16384, "drift": FLOOD},
        # the candidates of a flooded search, merged
        {"name": "cluster", "kind": "cluster", "ndm": 256, "nsamp": 1 << 20, "max_width": 4096, "baseline": 16384,
         "drift": FLOOD},
        # dedispersion of a short, few-channel chunk with rows of odd length
        {"name": "dedisp_small", "kind": "dedisp", "nchan": 256, "ndm": 128, "nsamp": 40001, "dm_max": 500.0,
         "tsamp": 98.304e-6},
        # dedispersion of the benchmark's chunk
        {"name": "dedisp_chunk", "kind": "dedisp", "nchan": 1024, "ndm": 1024, "nsamp": 1 << 18, "dm_max": 1000.0,
         "tsamp": 49.152e-6},
        # the benchmark's filterbank through both excision passes
        {"name": "rfi_chunk", "kind": "rfi", "nchan": 1024, "nsamp": 298529},
        # filterbank to clusters: excision, dedispersion, search, clustering
        {"name": "pipeline", "kind": "pipeline", "nchan": 512, "ndm": 256, "nsamp": 1 << 16, "dm_max": 700.0,
         "tsamp": 98.304e-6, "max_width": 1024, "baseline": 4096},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["search", "search", "search", "stream", "serve", "batch", "cluster", "dedisp", "dedisp", "rfi",
                       "pipeline"])
    case = {"kind": kind}
    if kind in ("search", "stream", "serve", "batch", "cluster"):
        case["max_width"] = 1 << rng.randint(5, 12)
        case["baseline"] = _log(rng, 1000, 20000)
        case["drift"] = rng.choice([FLOOD, SLOW])
    if kind == "search":
        nsamp = _log(rng, 5000, 1 << 19)
        samples = _log(rng, 1 << 19, 1 << 28)
        case.update(nsamp=nsamp, ndm=max(1, min(2048, samples // nsamp)), window=rng.randint(0, 1),
                    norm=rng.choice([0, 0, 1, 2]))
        case["blocks"] = 4 if case["ndm"] * nsamp < 1 << 22 else 1
    elif kind == "stream":
        case.update(nsamp=64 * _log(rng, 64, 2048), ndm=_log(rng, 64, 2048), gulps=2, norm=rng.randint(0, 1))
    elif kind == "serve":
        case.update(beams=rng.randint(2, 6), ndm=_log(rng, 128, 800), nsamp=64 * _log(rng, 128, 1024))
    elif kind == "batch":
        case.update(files=rng.randint(4, 16), ndm=_log(rng, 32, 256), nsamp=_log(rng, 1 << 14, 1 << 17))
    elif kind == "cluster":
        case.update(ndm=_log(rng, 32, 512), nsamp=_log(rng, 1 << 16, 1 << 18))
    elif kind == "dedisp":
        case.update(nchan=_log(rng, 64, 1024), ndm=_log(rng, 24, 1024), nsamp=_log(rng, 5000, 1 << 17),
                    dm_max=round(rng.uniform(100.0, 1000.0), 1), tsamp=rng.choice([49.152e-6, 64e-6, 98.304e-6]))
    elif kind == "rfi":
        case.update(nchan=_log(rng, 64, 1024), nsamp=_log(rng, 10000, 400000))
    else:
        case.update(nchan=_log(rng, 64, 512), ndm=_log(rng, 32, 256), nsamp=_log(rng, 1 << 14, 1 << 16),
                    dm_max=round(rng.uniform(100.0, 700.0), 1), tsamp=98.304e-6, max_width=1 << rng.randint(5, 10),
                    baseline=_log(rng, 1000, 4096))
    return case


# -- inputs

def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _series(g, ndm, nsamp, drift, max_width, t0=0):
    """Noise, drift and pulses of one block: FP32, integer-valued."""
    t = torch.arange(t0, t0 + nsamp, device="cuda", dtype=torch.float64)
    base = MU + torch.round(2.0 * SIGMA * torch.sin(2.0 * math.pi * t / drift))
    x = torch.randn((ndm, nsamp), generator=g, device="cuda")
    x.mul_(SIGMA).round_().add_(base.float())
    top = min(max_width, 1024, nsamp // 4)
    for _ in range(12):
        u = torch.rand(4, generator=g, device="cuda").tolist()
        w = max(1, int(math.exp(u[0] * math.log(max(1, top)))))
        row, at = int(u[1] * max(1, ndm - 2)), int(u[2] * (nsamp - w))
        x[row:row + 3, at:at + w] += round((6.0 + 44.0 * u[3]) * SIGMA / math.sqrt(w))
    return x


def _filterbank(g, nchan, nsamp, delays):
    """8-bit noise with dispersed pulses, broadband bursts and noisy channels."""
    x = torch.empty((nchan, nsamp), dtype=torch.uint8, device="cuda")
    sigma = torch.where(torch.rand(nchan, generator=g, device="cuda") < 0.02, 40.0, 6.0)
    for f in range(0, nchan, 64):
        part = torch.randn((min(64, nchan - f), nsamp), generator=g, device="cuda")
        part = part.mul_(sigma[f:f + 64, None]).add_(64.0).round_()
        x[f:f + 64] = part.clamp_(0.0, 255.0).to(torch.uint8)
    rows = torch.arange(nchan, device="cuda")

    def add(times, amp):
        keep = times < nsamp
        v = x[rows[keep], times[keep]].to(torch.int32) + amp
        x[rows[keep], times[keep]] = v.clamp_(max=255).to(torch.uint8)

    for k in range(8):
        u = torch.rand(3, generator=g, device="cuda").tolist()
        at, width = int(u[0] * nsamp * 0.9), 1 << int(u[1] * 8)
        amp = max(2, int(40.0 / math.sqrt(width)))
        trial = int(u[2] * delays.shape[0])
        for q in range(width):
            add(at + q + delays[trial], amp)
    for u in torch.rand(4, generator=g, device="cuda").tolist():
        at = int(u * (nsamp - 8))
        x[:, at:at + 4] = (x[:, at:at + 4].to(torch.int32) + 60).clamp_(max=255).to(torch.uint8)
    return x


def _delays(case):
    nchan, ndm = case["nchan"], case["ndm"]
    bw = (F_HI_MHZ - F_LO_MHZ) / nchan
    freqs = [F_HI_MHZ - bw * (f + 0.5) for f in range(nchan)]
    dms = [case["dm_max"] * d / max(1, ndm - 1) for d in range(ndm)]
    return sps.dedisp_delays(freqs, F_HI_MHZ, case["tsamp"], dms)


def _capacity(ndm, nsamp):
    """Records to hold: the flood of drift gives one in 100 to 130 samples."""
    return ndm * nsamp // 64 + 2048


def _buffers(capacity):
    return (torch.zeros((capacity, 4), dtype=torch.int32, device="cuda"),
            torch.zeros(1, dtype=torch.int32, device="cuda"))


def _plan(case, ndm, nsamp, capacity):
    plan = sps.Plan(ndm, nsamp, case["max_width"], case["baseline"], THRESH)
    plan.set(sps.ATTR_MAX_CANDS, capacity)
    if case.get("window"):
        plan.set(sps.ATTR_WINDOW, 1)
    if case.get("norm"):
        plan.set(sps.ATTR_NORM, case["norm"])
    return plan


def _shapes(case):
    """(ndm, nsamp) of each beam or file: uneven, around the case's."""
    n = case.get("beams") or case.get("files")
    step = 64 if case["kind"] == "serve" else 1
    got = []
    for i in range(n):
        ndm = max(1, case["ndm"] * (3 + (5 * i) % 7) // 6)
        nsamp = max(64, case["nsamp"] * (2 + (3 * i) % 5) // 4)
        got.append((ndm, (nsamp + 7 * i) // step * step))
    return got


def prepare(case, seed):
    g = _generator(seed)
    kind = case["kind"]
    if kind == "search":
        ndm, nsamp, n = case["ndm"], case["nsamp"], case["blocks"]
        cap = _capacity(ndm, nsamp)
        cands = torch.zeros((n, cap, 4), dtype=torch.int32, device="cuda")
        ncand = torch.zeros((n, 1), dtype=torch.int32, device="cuda")
        return {"kind": kind, "plan": _plan(case, ndm, nsamp, cap), "cands": cands, "ncand": ncand,
                "x": [_series(g, ndm, nsamp, case["drift"], case["max_width"]) for _ in range(n)]}
    if kind == "stream":
        ndm, nsamp, n = case["ndm"], case["nsamp"], case["gulps"]
        cap = _capacity(ndm, nsamp)
        plan = _plan(case, ndm, nsamp, cap)
        return {"kind": kind, "plan": plan, "stream": sps.Stream(plan), "out": [_buffers(cap) for _ in range(n)],
                "x": [_series(g, ndm, nsamp, case["drift"], case["max_width"], k * nsamp) for k in range(n)]}
    if kind == "serve":
        state = {"kind": kind, "batch": sps.Batch(), "plans": [], "streams": [], "x": [], "cands": [], "ncand": []}
        for i, (ndm, nsamp) in enumerate(_shapes(case)):
            cap = _capacity(ndm, nsamp)
            plan = _plan(dict(case, norm=i % 2), ndm, nsamp, cap)
            cands, ncand = _buffers(cap)
            state["plans"].append(plan)
            state["streams"].append(sps.Stream(plan))
            state["x"].append(_series(g, ndm, nsamp, case["drift"], case["max_width"]))
            state["cands"].append(cands)
            state["ncand"].append(ncand)
        return state
    if kind == "batch":
        items = []
        for ndm, nsamp in _shapes(case):
            x = _series(g, ndm, nsamp, case["drift"], case["max_width"])
            items.append((x, case["max_width"], case["baseline"], THRESH)
                         + _buffers(_capacity(ndm, nsamp)))
        return {"kind": kind, "batch": sps.Batch(), "items": items}
    if kind == "cluster":
        ndm, nsamp = case["ndm"], case["nsamp"]
        cap = _capacity(ndm, nsamp)
        cands, ncand = _buffers(cap)
        with _plan(case, ndm, nsamp, cap) as plan:
            plan.search(_series(g, ndm, nsamp, case["drift"], case["max_width"]), cands, ncand)
            n = int(ncand.item())
        return {"kind": kind, "cands": cands, "n": n, "clusterer": sps.Clusterer(cap)}
    if kind == "rfi":
        nchan, nsamp = case["nchan"], case["nsamp"]
        track = torch.arange(nchan, device="cuda")[None, :] * 30
        fil = _filterbank(g, nchan, nsamp, track)
        return {"kind": kind, "fil": fil, "masked": torch.empty_like(fil), "clean": torch.empty_like(fil),
                "stats": torch.empty((nchan, 3), dtype=torch.uint8, device="cuda")}
    table = _delays(case)
    nin = case["nsamp"] + int(table.max())
    fil = _filterbank(g, case["nchan"], nin, torch.from_numpy(table).cuda().long())
    state = {"kind": kind, "fil": fil, "dedisp": sps.Dedisperser(case["nchan"], nin, table)}
    state["block"] = state["dedisp"].alloc_out()
    if kind == "pipeline":
        cap = _capacity(case["ndm"], case["nsamp"])
        state.update(masked=torch.empty_like(fil), stats=torch.empty((case["nchan"], 3), dtype=torch.uint8,
                                                                     device="cuda"),
                     plan=_plan(case, case["ndm"], case["nsamp"], cap), out=_buffers(cap),
                     clusterer=sps.Clusterer(cap))
    return state


# -- one pass

def _keys(cands):
    """One integer per record that sorts by (row, sample, width)."""
    words = cands.view(torch.int64)  # sample | row << 32, width | snr << 32
    return (words[..., 0] << 13) | (words[..., 1] & 0x1FFF)


def _ordered(cands, ncand):
    """The candidates in a fixed order, the rest of the buffers' length filled
    up; with small buffers without waiting for the count."""
    cap = cands.shape[-2]
    snr = cands[..., 3].view(torch.float32)
    if cap > UNSORTED:
        n = int(ncand.item()) & 0xFFFFFFFF
        if n > cap:
            raise RuntimeError("candidate buffer too small")
        found, at = torch.sort(_keys(cands[:n]))
        keys, values = torch.full((cap,), INVALID, device="cuda"), torch.zeros(cap, device="cuda")
        keys[:n], values[:n] = found, snr[at]
        return {"ncand": ncand, "keys": keys, "snr": values}
    held = torch.arange(cap, device="cuda") < ncand
    keys, at = torch.sort(torch.where(held, _keys(cands), INVALID), dim=-1)
    return {"ncand": ncand, "keys": keys, "snr": torch.where(held, torch.gather(snr, -1, at), 0.0)}


def _clusters(state, cands, n):
    """The clusters in a fixed order, up to a fixed number of records."""
    k = state["clusterer"]
    out, nout = k.alloc_out(n)
    k.run(cands, n, *CLUSTER_TOL, out, nout)
    out = out[:int(nout.item())]
    best = out[:, 0].long() | (out[:, 1].long() << 32)
    rec = torch.zeros((cands.shape[0] // 4, 10), dtype=torch.int32, device="cuda")
    rec[:out.shape[0]] = out[torch.argsort((best << 13) | out[:, 2].long())]
    # record fields: sample, row, width | snr | members, sample extent, row extent
    return {"nout": nout, "best": rec[:, :3], "snr": rec[:, 3].view(torch.float32), "extent": rec[:, 4:9]}


def run(state):
    kind = state["kind"]
    if kind == "search":
        for i, x in enumerate(state["x"]):
            state["plan"].search(x, state["cands"][i], state["ncand"][i])
        if len(state["x"]) == 1:
            return _ordered(state["cands"][0], state["ncand"][0])
        if state["cands"].shape[1] > UNSORTED:
            return [_ordered(c, n) for c, n in zip(state["cands"], state["ncand"])]
        return _ordered(state["cands"], state["ncand"])
    if kind == "stream":
        for x, (cands, ncand) in zip(state["x"], state["out"]):
            state["stream"].push(x, cands, ncand, graph=True)
        return [_ordered(cands, ncand) for cands, ncand in state["out"]]
    if kind == "serve":
        state["batch"].push(state["streams"], state["x"], state["cands"], state["ncand"])
        return [_ordered(c, n) for c, n in zip(state["cands"], state["ncand"])]
    if kind == "batch":
        state["batch"].search(state["items"])
        return [_ordered(item[4], item[5]) for item in state["items"]]
    if kind == "cluster":
        return _clusters(state, state["cands"], state["n"])
    if kind == "rfi":
        sps.chan_mask(state["fil"], MASK_K, out=state["masked"], stats=state["stats"])
        sps.zero_dm(state["masked"], ZERO_OFFSET, out=state["clean"])
        return {"stats": state["stats"], "clean": state["clean"]}
    if kind == "dedisp":
        return state["dedisp"].run(state["fil"], out=state["block"])
    sps.chan_mask(state["fil"], MASK_K, out=state["masked"], stats=state["stats"])
    sps.zero_dm(state["masked"], ZERO_OFFSET, out=state["masked"])
    state["dedisp"].run(state["masked"], out=state["block"])
    cands, ncand = state["out"]
    state["plan"].search(state["block"], cands, ncand)
    found = {"stats": state["stats"], "block": state["block"], "cands": _ordered(cands, ncand)}
    found["clusters"] = _clusters(state, cands, min(int(ncand.item()), cands.shape[0]))
    return found


# -- what a pass cannot do without

def _search_work(ndm, nsamp, case):
    widths = int(math.log2(case["max_width"])) + 1
    # each sample read once, a candidate per few thousand samples written; per
    # sample and width a window sum (one subtraction) and a comparison
    found = 16 * ndm * nsamp // (128 if case["drift"] == FLOOD else 4096)
    return 4 * ndm * nsamp + found, 2.0 * widths * ndm * nsamp


def work(case):
    kind = case["kind"]
    if kind in ("search", "stream"):
        b, f = _search_work(case["ndm"], case["nsamp"], case)
        n = case.get("blocks") or case["gulps"]
        return {"bytes": n * b, "flops": n * f}
    if kind in ("serve", "batch"):
        each = [_search_work(ndm, nsamp, case) for ndm, nsamp in _shapes(case)]
        return {"bytes": sum(b for b, _ in each), "flops": sum(f for _, f in each)}
    if kind == "cluster":
        # candidates read once, a cluster record written for every 20 or so;
        # a handful of comparisons each
        n = case["ndm"] * case["nsamp"] // (128 if case["drift"] == FLOOD else 4096)
        return {"bytes": 18 * n, "flops": 20.0 * n}
    if kind == "rfi":
        n = case["nchan"] * case["nsamp"]
        return {"bytes": 2 * n + 3 * case["nchan"], "flops": 4.0 * n}
    nchan, ndm, nsamp = case["nchan"], case["ndm"], case["nsamp"]
    sweep = 4.148808e3 * case["dm_max"] * (F_LO_MHZ ** -2 - F_HI_MHZ ** -2) / case["tsamp"]
    fil = nchan * (nsamp + int(sweep))
    adds = float(nchan) * ndm * nsamp
    if kind == "dedisp":
        return {"bytes": fil + 4 * ndm * nsamp, "flops": adds}
    return {"bytes": fil + 4 * ndm * nsamp, "flops": adds + 4.0 * fil + 22.0 * ndm * nsamp}


# -- the same in 64 bits, in plain torch

MOST_SORTED = 4e9  # window samples of a block that are sorted in a few seconds


def _lower_median(v):
    return torch.sort(v, dim=-1).values[..., (v.shape[-1] - 1) // 2]


def _exact_stats(x, case):
    """Median and MAD of every 64-sample block's window."""
    ndm, nsamp = x.shape
    length, nb = case["baseline"], -(-nsamp // 64)
    lead = max(0, (length - 64) // 2) if case.get("window") else 0
    med = torch.empty((ndm, nb), dtype=torch.int32, device=x.device)
    mad = torch.empty_like(med)
    for k in range(nb):
        end = min(64 * k + 64, nsamp) + lead
        w = x[:, max(0, end - length):min(nsamp, end)]
        med[:, k] = _lower_median(w)
        mad[:, k] = _lower_median((w - med[:, k:k + 1]).abs())
    return med, mad


def _exact_search(x, case):
    """What _ordered() gives for one block, with its S/N in 64 bits."""
    ndm, nsamp = x.shape
    x = x.to(torch.int32)
    med, mad = _exact_stats(x, case)
    r = x - med.repeat_interleave(64, 1)[:, :nsamp]
    norm = case.get("norm", 0)
    if norm == 1:
        c = _lower_median(r)[:, None]
        mad[:] = _lower_median((r - c).abs())[:, None]
    total = torch.zeros((ndm, nsamp + 1), dtype=torch.int64, device=x.device)
    total[:, 1:] = torch.cumsum(r, 1, dtype=torch.int64)
    keys, found = [], []
    w = 1
    while w <= min(case["max_width"], nsamp):
        s = total[:, w:] - total[:, :total.shape[1] - w]
        if norm == 2:
            c = _lower_median(s)[:, None]
            scale = (1.482602218505602 * _lower_median((s - c).abs()).double())[:, None]
        else:
            at = (torch.arange(s.shape[1], device=x.device) + w // 2) // 64
            scale = 1.482602218505602 * mad[:, at].double() * math.sqrt(w)
        snr = torch.where(scale > 0, s.double() / scale, 0.0)
        above = snr > THRESH
        start = above.clone()
        start[:, 1:] &= ~above[:, :-1]
        runs = torch.cumsum(start.flatten(), 0)
        pos = above.flatten().nonzero()[:, 0]
        of, value = runs[pos] - 1, snr.flatten()[pos]
        count = int(runs[-1])
        best = torch.zeros(count, dtype=torch.float64, device=x.device).scatter_reduce_(0, of, value, "amax")
        first = torch.where(value == best[of], pos, INVALID)
        first = torch.full((count,), INVALID, device=x.device).scatter_reduce_(0, of, first, "amin")
        keys.append((((first // s.shape[1] << 32) | first % s.shape[1]) << 13) | w)
        found.append(best)
        w *= 2
    snr = torch.cat(found)[torch.argsort(torch.cat(keys))]
    return {"ncand": None, "keys": None, "snr": torch.cat([snr, snr.new_zeros(_capacity(ndm, nsamp) - snr.numel())])}


def _exact_dedisp(fil, table, nsamp):
    out = torch.zeros((table.shape[0], nsamp), dtype=torch.float64, device="cuda")
    table = torch.from_numpy(table).cuda().long()
    for f in range(fil.shape[0]):
        shifted = fil[f].as_strided((fil.shape[1] - nsamp + 1, nsamp), (1, 1), fil[f].storage_offset())
        out += shifted[table[:, f]]
    return out


def _exact_excised(fil):
    """Both excision passes: noisy channels replaced by their median, then the band's mean taken out."""
    x = fil.to(torch.int64)
    mu = _lower_median(fil).long()
    sigma = _lower_median((x - mu[:, None]).abs().to(torch.uint8)).long()
    mid = _lower_median(sigma)
    x = torch.where((sigma > mid + MASK_K * _lower_median((sigma - mid).abs()))[:, None], mu[:, None], x)
    level = torch.div(2 * x.sum(0) + x.shape[0], 2 * x.shape[0], rounding_mode="floor")
    return (x - level + ZERO_OFFSET).clamp_(0, 255).to(torch.uint8)


def exact(case, seed):
    kind, g = case["kind"], _generator(seed)

    def sortable(ndm, nsamp):
        return ndm * (nsamp // 64) * min(case["baseline"], nsamp) <= MOST_SORTED

    if kind == "search" and sortable(case["ndm"] * case["blocks"], case["nsamp"]):
        got = [_exact_search(_series(g, case["ndm"], case["nsamp"], case["drift"], case["max_width"]), case)
               for _ in range(case["blocks"])]
        if len(got) == 1:
            return got[0]
        if _capacity(case["ndm"], case["nsamp"]) > UNSORTED:
            return got
        return {"ncand": None, "keys": None, "snr": torch.stack([v["snr"] for v in got])}
    if kind == "batch" and sortable(sum(ndm * nsamp for ndm, nsamp in _shapes(case)) // 64, 64 * case["baseline"]):
        return [_exact_search(_series(g, ndm, nsamp, case["drift"], case["max_width"]), case)
                for ndm, nsamp in _shapes(case)]
    if kind in ("dedisp", "pipeline"):
        table = _delays(case)
        nin = case["nsamp"] + int(table.max())
        fil = _filterbank(g, case["nchan"], nin, torch.from_numpy(table).cuda().long())
        if kind == "dedisp":
            return _exact_dedisp(fil, table, case["nsamp"])
        block = _exact_dedisp(_exact_excised(fil), table, case["nsamp"])
        cands = _exact_search(block, case) if sortable(case["ndm"], case["nsamp"]) else None
        return {"stats": None, "block": block, "cands": cands, "clusters": None}
    # the large blocks, streams and beams have too many windows to sort; excision
    # and clustering return whole numbers and S/N values that they were given
    return None

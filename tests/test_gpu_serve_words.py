"""The pinned words that the serving executor copies candidate counts to: each
gulp has one of its own until its count is read, more than one block of them
when many gulps are in flight, and all come back."""
import numpy as np
import pytest

from paper_2512_00398_amd import serve

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch", [False, True])
def test_words_are_returned(batch):
    import torch
    beams, gulps, ndm, n = 5, 30, 2, 1024
    rng = np.random.default_rng(4)
    x = 1000.0 + np.round(rng.normal(0.0, 50.0, size=(beams, gulps, ndm, n)))
    for b in range(beams):
        for k in range(gulps):  # a different number of pulses in every gulp
            x[b, k, 0, 20:20 + 20 * ((7 * b + k) % 40):20] += 4000.0
    dev = torch.from_numpy(x.astype(np.float32)).cuda()
    spec = [serve.BeamSpec(ndm=ndm, nsamp=n, max_width=1, baseline_len=1000, snr_thresh=20.0)] * beams
    arr = serve.poisson_arrivals(spec, 1.0, seed=1, gulps_per_beam=gulps)
    ex = serve.GpuExecutor(lambda b, k: dev[b, k], nstreams=3, cand_cap=1 << 12, cand_slots=gulps, batch=batch)
    rep = serve.serve(spec, arr, ex, budget=1 << 40, compress=float("inf"))
    assert rep.max_inflight > 64
    for r in rep.records:
        assert r.ncand == (7 * r.beam + r.k) % 40, (r.beam, r.k, r.ncand)
    words = [w.data_ptr() for w in ex.words]
    assert len(words) == len(set(words)) and len(words) % 64 == 0 and len(words) >= rep.max_inflight

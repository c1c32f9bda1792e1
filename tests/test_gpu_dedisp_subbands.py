"""GPU parity of dedispersion over delay tables that share much, little or
nothing between neighbouring channels and trials (every tile shape and subband
width), at the edges of blocks, tiles and the filterbank. Exact integer sums."""
import numpy as np
import pytest

from oracle import dedisp_oracle as dd

pytestmark = pytest.mark.gpu


def table(kind, nchan, ndm, top, rng):
    f, d = np.arange(nchan), np.arange(ndm)[:, None]
    if kind == "shared":    # neighbouring trials and channels move together
        return np.floor(d * f * (top / max(1, (ndm - 1) * max(1, nchan - 1)))).astype(np.int64)
    if kind == "falling":   # delays fall with the trial and rise with the channel
        return np.floor((ndm - 1 - d) * f * (top / max(1, (ndm - 1) * max(1, nchan - 1)))).astype(np.int64)
    if kind == "wide":      # one pattern, trials far apart
        return np.broadcast_to(d * (top // max(1, ndm - 1)) + f % 3, (ndm, nchan)).astype(np.int64)
    return rng.integers(0, top + 1, size=(ndm, nchan))  # nothing shared


@pytest.mark.parametrize("kind", ["shared", "falling", "wide", "random"])
@pytest.mark.parametrize("nchan,ndm,nout,top", [
    (1, 1, 1, 0), (2, 3, 5, 3), (5, 33, 1008, 40), (7, 40, 1009, 700), (9, 17, 503, 250), (11, 8, 504, 255),
    (13, 64, 4033, 2000), (130, 65, 505, 90), (600, 21, 1500, 300), (1030, 34, 2017, 64)])
def test_tables(kind, nchan, ndm, nout, top):
    import torch
    from paper_2512_00398_amd import sps
    rng = np.random.default_rng(nchan * 7 + nout)
    tab = table(kind, nchan, ndm, top, rng)
    nin = nout + int(tab.max())
    fil = rng.integers(0, 256, size=(nchan, nin)).astype(np.uint8)
    if nchan == 600:
        fil[:] = 255  # the 16-bit sums at their largest
    print("dedisp table", kind, nchan, ndm, nout, int(tab.max()), flush=True)
    # the filterbank ends its buffer's used part: bytes after it must not matter
    buf = torch.full((nchan * nin + 64,), 255, dtype=torch.uint8, device="cuda")
    x = buf[:nchan * nin].view(nchan, nin)
    x.copy_(torch.from_numpy(fil))
    with sps.Dedisperser(nchan, nin, tab) as k:
        got = k.run(x)
        torch.cuda.synchronize()
    assert np.array_equal(got.cpu().numpy().astype(np.int64), dd.dedisperse(fil, tab))

"""GPU parity of the fused F+X on short calls: chunks down to one spectrum,
several dumps per round of workgroups, partials summed in segments, and the
filter history copied in the same launch (aligned and unaligned, calls shorter
than the filter).  Tolerance as for the other float32 F+X tests: 1e-5 of
sqrt(V_ii V_jj), the autos averaged over the dumps: the transform's rounding
follows the level of a channel, while a single spectrum's own |X|^2 can be
arbitrarily far below it."""

import numpy as np
import pytest

import synth
from oracle import pfb, xengine
from util import auto_scale

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_ant,N,spd,n_dump,off,acc", [
    (4, 4096, 1, 1, 0, False), (4, 4096, 2, 3, 1, False), (4, 4096, 33, 1, 0, True), (4, 1024, 1, 5, 0, True),
    (4, 1024, 45, 3, 3, False), (8, 1024, 3, 2, 0, False), (2, 4096, 1, 600, 0, False), (4, 512, 70, 9, 2, True),
    (2, 1024, 1000, 1, 0, False), (8, 2048, 2, 1, 0, False),
])
def test_short_calls(qc, n_ant, N, spd, n_dump, off, acc):
    import torch
    P = 4
    x = synth.generate(synth.array_spec(n_ant, N * (spd * n_dump + P - 1), 5 + N + spd, corr=0.3, max_lag=5))
    keep = (P - 1) * N
    hist, xs = np.ascontiguousarray(x[:, :keep]), np.ascontiguousarray(x[:, keep:])
    chans = np.arange(0, N // 2, max(1, N // 60))
    X = pfb.channelize(xs, N, P, chans=chans, hist=hist)
    ref = xengine.correlate_fast(X, spd)
    xd, hd = torch.from_numpy(xs).cuda(), torch.from_numpy(hist).cuda()
    ho = torch.zeros(n_ant * keep + off, dtype=torch.int8, device="cuda")
    nb = n_ant * (n_ant + 1) // 2
    vis = torch.ones((n_dump, nb, N // 2), dtype=torch.complex64, device="cuda") if acc else None
    out = qc.xcorrelate(xd, N, P, spd, hist=hd, hist_out=ho[off:].view(n_ant, keep), vis=vis, accumulate=acc)
    V = out.cpu().numpy()[:, :, chans] - (1.0 if acc else 0.0)
    scale = auto_scale(ref.mean(0, keepdims=True), n_ant)
    assert np.max(np.abs(V - ref) / scale) <= 1e-5
    assert np.array_equal(ho[off:].cpu().numpy().reshape(n_ant, keep), x[:, -keep:])


@pytest.mark.parametrize("n_spec", [1, 2, 3, 7])
def test_history_of_short_calls(qc, n_spec):
    """Fewer spectra than the filter has taps: part of the history stays."""
    import torch
    n_ant, N, P = 4, 1024, 4
    rng = np.random.default_rng(n_spec)
    x = rng.integers(-50, 51, (n_ant, N * (P - 1 + n_spec))).astype(np.int8)
    keep = (P - 1) * N
    hd, xd = torch.from_numpy(x[:, :keep].copy()).cuda(), torch.from_numpy(x[:, keep:].copy()).cuda()
    ho = torch.zeros_like(hd)
    qc.xcorrelate(xd, N, P, n_spec, hist=hd, hist_out=ho)
    assert np.array_equal(ho.cpu().numpy(), x[:, -keep:])
    qc.xcorrelate(xd, N, P, n_spec, hist=None, hist_out=ho)
    want = np.concatenate([np.zeros((n_ant, keep), np.int8), x[:, keep:]], 1)[:, -keep:]
    assert np.array_equal(ho.cpu().numpy(), want)

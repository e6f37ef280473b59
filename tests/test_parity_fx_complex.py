"""GPU parity of the fused F+X of complex words: every fused shape and word,
runs of one spectrum up to several, run counts that do and do not divide into
the blocks of an even/odd pair, carried history, user taps, accumulation.
Within 1e-5 of sqrt(V_ii V_jj) of the float64 oracle, the autos averaged over
the dumps; the filter history exact."""

import numpy as np
import pytest

from oracle import pfb, xengine
from util import auto_scale

pytestmark = pytest.mark.gpu


def _words(word, n_ant, n_samp, seed):
    """Complex Gaussian words with a component common to all antennas."""
    rng = np.random.default_rng(seed)
    sigma, top, dt = (1200.0, 8191, np.int16) if word == "ci16" else (16.0, 127, np.int8)
    common = rng.normal(size=(n_samp, 2)) * sigma * 0.55
    x = rng.normal(size=(n_ant, n_samp, 2)) * sigma * 0.83 + common
    return np.clip(np.round(x), -top, top).astype(dt)


@pytest.mark.parametrize("word", ["ci8", "ci16"])
@pytest.mark.parametrize("n_ant,N,spd,n_dump,mode", [
    (4, 4096, 1, 1, "plain"), (4, 4096, 9, 2, "hist"), (4, 4096, 3, 5, "taps"), (4, 4096, 40, 1, "acc"),
    (4, 2048, 7, 3, "hist"), (4, 2048, 1, 2, "taps"), (4, 1024, 33, 2, "hist"), (4, 1024, 5, 1, "acc"),
    (2, 4096, 6, 3, "hist"), (2, 4096, 2, 1, "taps"),
])
def test_complex_fused(qc, word, n_ant, N, spd, n_dump, mode):
    import torch
    P = 4
    keep = (P - 1) * N
    x = _words(word, n_ant, N * (spd * n_dump + 1) + keep, seed=N + spd)  # one spectrum beyond the dumps
    h, xs = np.ascontiguousarray(x[:, :keep]), np.ascontiguousarray(x[:, keep:])
    taps = np.random.default_rng(N).normal(size=P * N).astype(np.float32) if mode == "taps" else None
    carry = mode in ("hist", "acc")
    chans = np.concatenate([np.arange(0, N, max(1, N // 40)), [1, N // 2 - 1, N // 2, N // 2 + 1, N - 1]])
    iq = lambda v: v[..., 0].astype(np.int64) + 1j * v[..., 1].astype(np.int64)  # noqa: E731
    X = pfb.channelize_complex(iq(xs), N, P, chans=chans, hist=iq(h) if carry else None,
                               taps=None if taps is None else taps.astype(np.float64))
    ref = xengine.correlate_fast(X, spd)
    hd = torch.from_numpy(h).cuda() if carry else None
    ho = torch.zeros_like(torch.from_numpy(h)).cuda()
    nb = n_ant * (n_ant + 1) // 2
    vis = torch.ones((n_dump, nb, N), dtype=torch.complex64, device="cuda") if mode == "acc" else None
    out = qc.xcorrelate_ex(torch.from_numpy(xs).cuda(), N, P, spd, hist=hd, hist_out=ho, vis=vis,
                           accumulate=mode == "acc", taps=None if taps is None else torch.from_numpy(taps).cuda())
    V = out.cpu().numpy()[:, :, chans] - (1.0 if mode == "acc" else 0.0)
    assert np.max(np.abs(V - ref) / auto_scale(ref.mean(0, keepdims=True), n_ant)) <= 1e-5
    autos = [a * n_ant - a * (a - 1) // 2 for a in range(n_ant)]
    assert not np.any(out.cpu().numpy()[:, autos].imag - 0.0)
    full = np.concatenate([h if carry else np.zeros_like(h), xs], axis=1)
    assert np.array_equal(ho.cpu().numpy(), full[:, -keep:])

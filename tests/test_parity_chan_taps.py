"""GPU parity of the register-ring F-engine with any prototype: tap counts of
1 to 8 (those under 4 and between 5 and 8 run on zero taps), every size it
takes, antenna counts that leave part of a group empty, runs of one spectrum
and more, carried history.  Channelised voltages within 1e-5 of the channel
rms of the float64 oracle (as for the other F-engines) and within 5e-6 of the
plain kernel; the history exact."""

import numpy as np
import pytest

from oracle import pfb

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,n_ant,P,n_spec", [
    (1024, 1, 1, 3), (1024, 5, 8, 40), (1024, 4, 3, 300), (2048, 13, 8, 21), (2048, 3, 5, 9), (2048, 2, 2, 70),
    (4096, 7, 8, 12), (4096, 4, 6, 1), (4096, 3, 4, 90), (4096, 2, 1, 5), (8192, 3, 4, 7), (8192, 1, 3, 4),
    (8192, 2, 7, 3),
])
@pytest.mark.parametrize("carry", [False, True])
def test_any_prototype(qc, N, n_ant, P, n_spec, carry):
    import torch
    rng = np.random.default_rng(N + 10 * P + n_ant)
    x = rng.integers(-100, 101, (n_ant, N * n_spec)).astype(np.int8)
    taps = rng.normal(size=P * N).astype(np.float32)
    keep = (P - 1) * N
    carry = carry and keep > 0
    hist = rng.integers(-100, 101, (n_ant, keep)).astype(np.int8) if carry else None
    hd = torch.from_numpy(hist).cuda() if carry else None
    ho = torch.empty_like(hd) if carry else None
    xd, td = torch.from_numpy(x).cuda(), torch.from_numpy(taps).cuda()
    chans = np.arange(0, N // 2, max(1, N // 64))
    ref = pfb.channelize(x, N, P, taps=taps.astype(np.float64), hist=hist, chans=chans)
    rms = np.sqrt(np.mean(np.abs(ref) ** 2))
    out, _ = qc.pfb_channelize(xd, N, P, taps=td, hist=hd, hist_out=ho)
    got = out.cpu().numpy()
    assert np.max(np.abs(got[:, :, chans] - ref)) <= 1e-5 * rms
    prev = qc.channelize_variant()
    try:
        qc.channelize_variant(1)
        plain, _ = qc.pfb_channelize(xd, N, P, taps=td, hist=hd)
    finally:
        qc.channelize_variant(prev)
    assert np.max(np.abs(got - plain.cpu().numpy())) <= 5e-6 * rms
    if carry:
        assert np.array_equal(ho.cpu().numpy(), np.concatenate([hist, x], 1)[:, -keep:])


@pytest.mark.parametrize("word", ["i16", "ci8", "ci16"])
@pytest.mark.parametrize("N,P", [(1024, 2), (2048, 4), (4096, 3), (8192, 4)])
def test_any_prototype_of_other_words(qc, word, N, P):
    import torch
    n_ant, n_spec = 3, 6
    rng = np.random.default_rng(N + P)
    top = 100 if word == "ci8" else 8000
    shape = (n_ant, N * n_spec) + ((2,) if word.startswith("c") else ())
    x = rng.integers(-top, top + 1, shape).astype(np.int8 if word == "ci8" else np.int16)
    taps = rng.normal(size=P * N).astype(np.float32)
    out, _ = qc.pfb_channelize_ex(torch.from_numpy(x).cuda(), N, P, taps=torch.from_numpy(taps).cuda())
    got = out.cpu().numpy()
    n_chan = got.shape[2]
    chans = np.arange(0, n_chan, max(1, n_chan // 40))
    t64 = taps.astype(np.float64)
    if word.startswith("c"):
        ref = pfb.channelize_complex(x[..., 0].astype(np.int64) + 1j * x[..., 1], N, P, taps=t64, chans=chans)
    else:
        ref = pfb.channelize(x, N, P, taps=t64, chans=chans)
    assert np.max(np.abs(got[:, :, chans] - ref)) <= 1e-5 * np.sqrt(np.mean(np.abs(ref) ** 2))

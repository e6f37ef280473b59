"""GPU parity over runs of several spectra per workgroup: the loops of the fused
F+X (every word and shape) and of the ring F-engine (any prototype), whose sums,
blocks and buffers are carried from one spectrum to the next.  Each test looks up
the run length it gets.  Against the float64 oracle on a few channels: voltages
within 1e-5 of the channel rms, visibilities within 1e-5 of sqrt(V_ii V_jj)."""

import numpy as np
import pytest

from oracle import pfb, xengine
from util import vis_err

pytestmark = pytest.mark.gpu

SAMPLE = {"i8": 0, "i16": 1, "ci8": 2, "ci16": 3}


def _words(word, n_ant, n_samp, seed):
    rng = np.random.default_rng(seed)
    sigma, top, dt = (1200.0, 8191, np.int16) if word.endswith("16") else (16.0, 127, np.int8)
    parts = (2,) if word.startswith("c") else ()
    common = rng.normal(size=(n_samp,) + parts).astype(np.float32) * np.float32(sigma * 0.55)
    x = np.empty((n_ant, n_samp) + parts, dt)
    for a in range(n_ant):
        v = rng.standard_normal((n_samp,) + parts, np.float32) * np.float32(sigma * 0.83) + common
        x[a] = np.clip(np.round(v), -top, top)
    return x


def _oracle(word, x, N, P, chans, hist=None, taps=None):
    """X[a, m, k], one antenna at a time (the frames of all would fill memory)."""
    out = []
    for a in range(x.shape[0]):
        v, h = x[a:a + 1], None if hist is None else hist[a:a + 1]
        if word.startswith("c"):
            iq = lambda w: w[..., 0].astype(np.float64) + 1j * w[..., 1]  # noqa: E731
            out.append(pfb.channelize_complex(iq(v), N, P, taps=taps, hist=None if h is None else iq(h), chans=chans))
        else:
            out.append(pfb.channelize(v, N, P, taps=taps, hist=h, chans=chans))
    return np.concatenate(out)


@pytest.fixture
def ring_always(qc):
    qc.lib().qc_channelize_ring_always(1)
    yield
    qc.lib().qc_channelize_ring_always(0)


FUSED = [("i8", 4, 4096), ("i8", 2, 4096), ("i8", 4, 1024), ("i8", 8, 1024), ("i8", 4, 2048)] + [
    (w, a, n) for w in ("i16", "ci8", "ci16") for a, n in ((4, 4096), (2, 4096), (4, 1024), (4, 2048))]


@pytest.mark.parametrize("word,n_ant,N,run", [c + (r,) for c in FUSED for r in (2, 3)] +
                         [(w, 4, 4096, 8) for w in SAMPLE] + [("i8", 4, 1024, 9), ("ci8", 4, 2048, 9)])
def test_fused(qc, word, n_ant, N, run):
    import torch
    P, n_dump, s = 4, 2, SAMPLE[word]
    length = qc.lib().qc_fx_run_spectra
    spd = next(m for m in range(run, 20000) if length(s, N, n_ant, n_dump, m) == run) + 1
    assert length(s, N, n_ant, n_dump, spd) == run  # runs of this length and of one more
    keep = (P - 1) * N
    x = _words(word, n_ant, keep + N * spd * n_dump, N + run)
    hist, x = np.ascontiguousarray(x[:, :keep]), np.ascontiguousarray(x[:, keep:])
    n_chan = N if word.startswith("c") else N // 2
    chans = np.array([0, 1, 77, n_chan // 2 + 3, n_chan - 1])
    ref = xengine.correlate_fast(_oracle(word, x, N, P, chans, hist), spd)
    call = qc.xcorrelate if word == "i8" else qc.xcorrelate_ex
    V = call(torch.from_numpy(x).cuda(), N, P, spd, hist=torch.from_numpy(hist).cuda())
    assert vis_err(V.cpu().numpy()[:, :, chans], ref, n_ant) <= 1e-5


@pytest.mark.parametrize("word,n_ant,N,P", [
    ("i8", 4, 1024, 4), ("i8", 5, 1024, 8), ("i8", 3, 1024, 3), ("i8", 13, 2048, 8), ("i8", 4, 2048, 2),
    ("i8", 7, 4096, 8), ("i8", 4, 4096, 4), ("i8", 5, 4096, 1), ("i8", 3, 8192, 4), ("i8", 2, 8192, 3),
    ("i16", 4, 1024, 4), ("i16", 6, 4096, 3), ("ci8", 3, 2048, 4), ("ci8", 2, 8192, 2), ("ci16", 3, 1024, 3),
    ("ci16", 2, 4096, 4),
])
@pytest.mark.parametrize("run", [1, 2, 3, 9])
def test_ring(qc, ring_always, word, n_ant, N, P, run):
    import torch
    s = SAMPLE[word]
    length = qc.lib().qc_channelize_run_spectra
    n_spec = next(m for m in range(run, 20000) if length(s, N, n_ant, m) == run)
    keep = (P - 1) * N
    x = _words(word, n_ant, keep + N * n_spec, N + P)
    hist, x = np.ascontiguousarray(x[:, :keep]), np.ascontiguousarray(x[:, keep:])
    taps = np.random.default_rng(N + P).normal(size=P * N).astype(np.float32)
    n_chan = N if word.startswith("c") else N // 2
    chans = np.array([1, n_chan // 3, n_chan - 1])
    ref = _oracle(word, x, N, P, chans, hist if keep else None, taps.astype(np.float64))
    hd = torch.from_numpy(hist).cuda() if keep else None
    out, _ = qc.pfb_channelize_ex(torch.from_numpy(x).cuda(), N, P, taps=torch.from_numpy(taps).cuda(), hist=hd)
    got = out[:, :, torch.from_numpy(chans).cuda()].cpu().numpy()
    assert np.max(np.abs(got - ref)) <= 1e-5 * np.sqrt(np.mean(np.abs(ref) ** 2))


@pytest.mark.parametrize("word,n_ant,N,P,n_spec,ring", [
    ("i8", 4, 4096, 4, 1024, True), ("i8", 1, 1024, 1, 16384, False), ("i8", 4, 1024, 1, 64, False),
    ("i8", 13, 2048, 8, 1531, True), ("ci16", 4, 4096, 4, 1024, True), ("ci16", 13, 1024, 1, 157, False),
    ("i8", 2, 8192, 1, 256, False),
])
def test_the_choice_of_kernel(qc, word, n_ant, N, P, n_spec, ring):
    """By default the kernel that is the faster one by a clear margin runs: the
    spectra are that kernel's, to the bit."""
    import torch
    x = torch.from_numpy(_words(word, n_ant, N * n_spec, 5)).cuda()
    t = torch.from_numpy(np.random.default_rng(P).normal(size=P * N).astype(np.float32)).cuda()
    got, _ = qc.pfb_channelize_ex(x, N, P, taps=t)
    try:
        if ring:
            qc.lib().qc_channelize_ring_always(1)
        else:
            qc.channelize_variant(1)
        ref, _ = qc.pfb_channelize_ex(x, N, P, taps=t)
    finally:
        qc.lib().qc_channelize_ring_always(0)
        qc.channelize_variant(0)
    assert torch.equal(got, ref)

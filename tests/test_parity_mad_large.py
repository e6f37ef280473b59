"""GPU parity: MAD of large populations, whose windows come from a sample.

Masks and thresholds are bit-exact with the oracle at the edges of the route
(36864 elements), with rows that do or do not divide into fours, unaligned
planes, both contiguous populations, and on inputs where a sample misleads or
the lists overflow, so that the selection from the start takes over.
"""

import numpy as np
import pytest

from oracle import mad

pytestmark = pytest.mark.gpu


def _check(qc, v, sigma, pop, off=0):
    import torch
    m_ref, T_ref = mad.mad_flag(v, sigma, pop)
    buf = torch.zeros(v.size + off, dtype=torch.complex64, device="cuda")
    d = buf[off:].view(v.shape)
    d.copy_(torch.from_numpy(v).cuda())
    m, T = qc.mad_flag(d, sigma, pop)
    assert np.array_equal(T.cpu().numpy(), T_ref)
    assert np.array_equal(m.cpu().numpy(), m_ref)


def _noise(shape, seed):
    rng = np.random.default_rng(seed)
    return (rng.normal(size=shape) + 1j * rng.normal(size=shape)).astype(np.complex64)


@pytest.mark.parametrize("shape,pop,off", [
    ((1, 2, 36864), 0, 0), ((1, 3, 36868), 0, 0), ((1, 2, 36865), 0, 0), ((39, 2, 1001), 0, 0),
    ((20, 3, 2048), 0, 1), ((3, 2, 40000), 2, 0), ((2, 2, 36870), 2, 1), ((5, 1, 98304), 0, 0),
])
@pytest.mark.parametrize("sigma", [0.0, 3.0])
def test_large_populations(qc, shape, pop, off, sigma):
    _check(qc, _noise(shape, sum(shape)), sigma, pop, off)


def test_uneven_plane(qc):
    """A steep bandpass, a drifting gain, strong lines and bursts: the sample
    sees every channel and integration alike."""
    shape = (128, 2, 2048)
    rng = np.random.default_rng(5)
    v = _noise(shape, 6) * (0.01 + np.sin(np.linspace(0, 3.1, 2048))) * np.linspace(0.2, 5, 128)[:, None, None]
    v *= 1 + 40 * (rng.uniform(size=2048) < 0.03)
    v *= 1 + 20 * (rng.uniform(size=(128, 1, 1)) < 0.05)
    _check(qc, v.astype(np.complex64), 5.0, 0)


@pytest.mark.parametrize("fill", ["zero", "mostly", "half", "blocks", "two"])
def test_populations_a_sample_cannot_bound(qc, fill):
    shape = (64, 3, 2048)
    v = _noise(shape, 9)
    if fill == "zero":
        v[:, 1] = 0
    elif fill == "mostly":
        v[:48] = 0
    elif fill == "half":
        v[:32] = 0
    elif fill == "blocks":  # one element of four carries the signal
        v.reshape(64, 3, 512, 4)[..., 1:] *= np.float32(1e-3)
    else:
        v = np.where(np.arange(2048) % 2 == 0, np.complex64(3 + 4j), np.complex64(1)) * np.ones(shape, np.complex64)
    _check(qc, v.astype(np.complex64), 5.0, 0)


def test_not_finite_amplitudes(qc):
    """Amplitudes that are no number order above infinity and are not flagged."""
    import torch
    v = _noise((24, 2, 2048), 3)
    v[3, 0, ::7] = np.inf
    w = v.copy()
    w[5, 0, ::5] = np.nan
    v[5, 0, ::5] = np.inf
    with np.errstate(invalid="ignore"):
        m_ref, T_ref = mad.mad_flag(v, 5.0, 0)
    m_ref = np.array(m_ref)
    m_ref[5, 0, ::5] = 0
    m, T = qc.mad_flag(torch.from_numpy(w).cuda(), 5.0, 0)
    assert np.array_equal(T.cpu().numpy(), T_ref)
    assert np.array_equal(m.cpu().numpy(), m_ref)


def test_normalised_input_over_its_range(qc):
    """The flagger's input sign(r) log1p|r| over 16 decades of r, to one unit
    of float32 of the float64 value (one rounding each): rows that are not a
    multiple of a block, a constant plane and infinite amplitudes."""
    import torch
    from oracle import cnn
    rng = np.random.default_rng(4)
    n_time, n_chan = 8, 1030
    v = _noise((n_time, 3, n_chan), 12)
    v[:, 0] += 1000.0
    v[0, 0, :600] += (10.0 ** rng.uniform(-9, 9, 600)).astype(np.float32)
    v[:, 1] = 3 + 4j
    v[1, 2, 5] = np.inf
    with np.errstate(invalid="ignore"):
        ref = np.asarray(cnn.normalize(v), np.float64)
    x = qc.cnn_normalize(torch.from_numpy(v).cuda()).cpu().numpy()
    fin = np.isfinite(ref)
    assert np.array_equal(fin, np.isfinite(x))
    assert np.all(np.abs(x[fin] - ref[fin]) <= 2.0 ** -23 * np.abs(ref[fin]))


@pytest.mark.parametrize("off", [0, 1])
def test_open_populations_beside_closed_ones(qc, off):
    """More populations than compute units, some left open: zero, mostly zero,
    a few values that repeat, a group of equal amplitudes at the median and one
    at the threshold."""
    import torch
    n_base = torch.cuda.get_device_properties(0).multi_processor_count + 44
    v = _noise((37, n_base, 1000 + 4 * off), 21)
    v[:, 1::7] = 0
    v[:30, 2::7] = 0
    v[:, 3::7] = np.round(2 * v[:, 3::7].real) / 2
    a = np.abs(v[:, 4::7])
    v[:, 4::7][(a > 0.9) & (a < 1.4)] = np.complex64(1.2)
    med = np.median(a, axis=(0, 2), keepdims=True)
    top = med + 3 * 1.4826 * np.median(np.abs(a - med), axis=(0, 2), keepdims=True)
    v[:, 5::7][:, :a.shape[1], :90] = top[:, :v[:, 5::7].shape[1]].astype(np.complex64)
    _check(qc, v, 3.0, 0, off)


@pytest.mark.parametrize("shape,pop,off", [
    ((1, 3, 41996), 0, 0), ((42, 2, 1000), 0, 0), ((59, 2, 1001), 0, 0), ((60, 2, 1001), 0, 0), ((30, 3, 2048), 0, 1),
    ((1, 2, 59999), 2, 0), ((2, 1, 60003), 2, 0), ((2, 130, 36865), 2, 1), ((2, 150, 36868), 2, 0),
    ((28, 3, 2048), 0, 0), ((28, 300, 1336), 0, 0),
])
def test_edges_of_the_route(qc, shape, pop, off):
    """Few populations from 42000 elements, read one by one from 60000, and more
    populations than compute units from 36865."""
    _check(qc, _noise(shape, sum(shape)), 4.0, pop, off)


def test_a_sample_that_misled(qc):
    """Windows that miss: the sample takes elements of one pattern, the rest of the
    population differs, so the amplitudes are formed by the last step."""
    n = 65536
    n4, strata = n // 4, 3072
    g = np.arange(strata, dtype=np.int64)
    g0, g1 = g * n4 // strata, (g + 1) * n4 // strata
    h = (g.astype(np.uint32) * np.uint32(2654435761)) >> np.uint32(8)
    at = g0 + h.astype(np.int64) % (g1 - g0)
    v = _noise((1, 2, n), 17)
    v[0, 0] *= np.float32(50)
    quads = v[0, 0].reshape(n4, 4)
    quads[at] /= np.float32(50)
    _check(qc, v, 5.0, 0)

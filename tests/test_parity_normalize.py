"""GPU parity of the flagger's input at every row length the kernel splits
differently: rows that share a block (up to 512 channels, in groups of 1 to 128
lanes), a block per row and several; integration counts that are fewer and more
than the rows of a block; more rows than a launch has blocks.  Within one unit
of float32 of the float64 value (one rounding each)."""

import numpy as np
import pytest

from oracle import cnn

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_time", [1, 7, 256, 301])
@pytest.mark.parametrize("n_chan", [1, 3, 4, 5, 32, 33, 255, 256, 257, 512, 513, 1024, 1025, 2100])
def test_row_lengths(qc, n_time, n_chan):
    import torch
    rng = np.random.default_rng(n_time * 4096 + n_chan)
    shape = (n_time, 5, n_chan)
    v = (rng.normal(size=shape) + 1j * rng.normal(size=shape)).astype(np.complex64)
    ref = np.asarray(cnn.normalize(v), np.float64)
    x = qc.cnn_normalize(torch.from_numpy(v).cuda()).cpu().numpy()
    assert np.all(np.abs(x - ref) <= 2.0 ** -23 * np.abs(ref))


def test_more_rows_than_a_launch_has_blocks(qc):
    """2^24 + 16 rows of 4 channels; the float64 values by torch."""
    import torch
    n_time, n_base, n_chan = (1 << 20) + 1, 16, 4
    g = torch.Generator(device="cuda")
    g.manual_seed(8)
    v = torch.view_as_complex(torch.randn((n_time, n_base, n_chan, 2), generator=g, device="cuda"))
    x = qc.cnn_normalize(v)
    k = n_time * n_chan
    for b in range(n_base):
        a = torch.view_as_real(v[:, b].contiguous()).double().square().sum(-1).sqrt().float().double().flatten()
        s = a.sort().values
        med = 0.5 * (s[(k - 1) // 2] + s[k // 2])
        s = (a - med).abs().sort().values
        r = (a - med) / (1.4826 * 0.5 * (s[(k - 1) // 2] + s[k // 2]))
        ref = torch.sign(r) * torch.log1p(r.abs())
        assert bool(((x[b].flatten().double() - ref).abs() <= 2.0 ** -23 * ref.abs()).all())


def test_rounding_of_small_deviations(qc):
    """Deviations of 2^-10 to 2^-9 scales, whose bits 1 + r cannot hold: a float64
    error of 1e-15 moves the float32 rounding of 1e7 values 0.2 times (two
    elements of 2e7 are allowed), one of 1e-13 at 2^-10 about ten times."""
    import torch
    rng = np.random.default_rng(1)
    n_base, k = 200, 49800
    u = rng.uniform(2.0 ** -10, 2.0 ** -9, (n_base, k)) * rng.choice([-1, 1], (n_base, k)) * 1.4826
    a = np.concatenate([np.zeros((n_base, 25050)), 1 + u, np.ones((n_base, 100)), 2 * np.ones((n_base, 25050))], 1)
    a *= rng.uniform(0.5, 1.0, n_base)[:, None]
    v = np.ascontiguousarray(a.astype(np.float32).reshape(n_base, 100, 1000).transpose(1, 0, 2)).astype(np.complex64)
    x = qc.cnn_normalize(torch.from_numpy(v).cuda()).cpu().numpy()
    assert np.sum(x != np.asarray(cnn.normalize(v)).astype(np.float32)) <= 2


def test_scales_out_of_range(qc):
    """Infinite medians and deviations, and amplitudes that are no number."""
    import torch
    rng = np.random.default_rng(2)
    v = (rng.normal(size=(16, 4, 64)) + 1j * rng.normal(size=(16, 4, 64))).astype(np.complex64)
    v[:6, 0] = np.inf          # finite scale
    v[:9, 1] = np.inf          # infinite median
    v[2, 2, 3] = np.nan
    v[:, 3] *= np.float32(1e-38)
    with np.errstate(invalid="ignore"):
        ref = np.asarray(cnn.normalize(v), np.float64)
    x = qc.cnn_normalize(torch.from_numpy(v).cuda()).cpu().numpy()
    assert np.array_equal(np.isnan(x), np.isnan(ref)) and np.array_equal(np.isinf(x), np.isinf(ref))
    fin = np.isfinite(ref)
    assert np.all(np.abs(x[fin] - ref[fin]) <= 2.0 ** -23 * np.abs(ref[fin]))

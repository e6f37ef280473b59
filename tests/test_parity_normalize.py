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

"""GPU parity of the two ways conjugate samples reach the grid: added with the
samples (few) and by a pass over the finished sums (many), either side of the
line between them.  A cell of k samples is within k 2^-24 of its sum of
magnitudes; the Hermitian halves agree to the same."""

import numpy as np
import pytest

from oracle import imaging

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,k", [(64, 1), (64, 3000), (64, 45184), (64, 45185), (256, 47104), (256, 47108), (128, 60000)])
@pytest.mark.parametrize("skip", [0, 1])
def test_conjugates(qc, n, k, skip):
    import torch
    cell = 1e-3
    rng = np.random.default_rng(n + k)
    u, v = (rng.uniform(-0.55, 0.55, (2, k + skip)) / cell).astype(np.float32)
    u[::7] = 0
    v[::7] = 0                                   # the cell that is its own mirror
    vis = (rng.normal(size=k + skip) + 1j * rng.normal(size=k + skip)).astype(np.complex64)
    d = [torch.from_numpy(a).cuda()[skip:] for a in (u, v, vis)]
    g, ws = qc.image_grid(*d, n, cell)
    u, v, vis = u[skip:], v[skip:], vis[skip:]
    one = np.ones(k, np.float32)
    G_ref, W_ref = imaging.grid_nearest(u, v, vis, one, n, cell)
    mag, _ = imaging.grid_nearest(u, v, np.abs(vis), one, n, cell)
    cnt, _ = imaging.grid_nearest(u, v, one, one, n, cell)
    assert np.all(np.abs(g.cpu().numpy() - G_ref) <= (cnt.real + 2) * 2.0 ** -24 * 2 * mag.real)
    assert ws.item() == pytest.approx(W_ref, rel=1e-12)

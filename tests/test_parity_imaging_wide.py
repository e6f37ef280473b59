"""GPU parity of CLEAN over many workgroups and of gridding by runs.

CLEAN: components and residual bit-identical to the oracle at every launch
shape (one workgroup, 4, 16 and 64 with the residual in registers, 64 with it
in memory), on inputs whose values repeat, so that peaks tie across
workgroups.  Gridding: runs of samples in one cell that begin and end
anywhere, sample counts that fill neither a thread nor a wave, and unaligned
arrays; a cell of k samples is within k 2^-24 of its sum of magnitudes.
"""

import numpy as np
import pytest

from oracle import imaging

pytestmark = pytest.mark.gpu


def _dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _clean_input(n, seed):
    rng = np.random.default_rng(seed)
    D = (rng.integers(-64, 65, (n, n)) / 64).astype(np.float32)
    P = (rng.integers(-16, 17, (n, n)) / 64).astype(np.float32)
    P[n // 2, n // 2] = 1.0
    return D, P


@pytest.mark.parametrize("n,iters", [(2, 5), (32, 60), (64, 70), (128, 70), (256, 65), (512, 30), (1024, 20),
                                     (2048, 8)])
def test_clean_ties_across_workgroups(qc, n, iters):
    D, P = _clean_input(n, n)
    pix_r, flux_r, R_r = imaging.hogbom(D, P, 0.3, 0.0, iters)
    res = _dev(D)
    pix, flux = qc.image_clean(res, _dev(P), 0.3, 0.0, iters)
    assert np.array_equal(pix.cpu().numpy().astype(np.int64), pix_r)
    assert np.array_equal(flux.cpu().numpy(), flux_r)
    assert np.array_equal(res.cpu().numpy(), R_r)


def test_clean_on_two_streams(qc):
    import torch
    made = [_clean_input(n, 7 * n) for n in (256, 512)]
    ref = [imaging.hogbom(D, P, 0.2, 0.0, 40) for D, P in made]
    ins = [(_dev(D), _dev(P)) for D, P in made]
    streams = [torch.cuda.Stream() for _ in ins]
    torch.cuda.synchronize()
    got = []
    for (d, p), s in zip(ins, streams):
        with torch.cuda.stream(s):
            got.append(qc.image_clean(d, p, 0.2, 0.0, 40))
    torch.cuda.synchronize()
    for (d, _), (pix, flux), (pix_r, flux_r, R_r) in zip(ins, got, ref):
        assert np.array_equal(pix.cpu().numpy(), pix_r)
        assert np.array_equal(flux.cpu().numpy(), flux_r)
        assert np.array_equal(d.cpu().numpy(), R_r)


def test_clean_not_a_number_is_no_peak(qc):
    D, P = _clean_input(128, 3)
    D[5, 7] = np.nan
    D[90, 1] = np.float32(3.0)
    res = _dev(D)
    pix, flux = qc.image_clean(res, _dev(P), 0.5, 0.1, 1)
    assert pix.cpu().numpy().tolist() == [90 * 128 + 1]
    assert flux.cpu().numpy().tolist() == [1.5]


@pytest.mark.parametrize("k,skip,weighted", [(1, 0, False), (3, 0, True), (255, 1, True), (1026, 0, False),
                                             (5000, 3, True), (20001, 0, True)])
def test_grid_runs(qc, k, skip, weighted):
    n, cell = 128, 1e-3
    rng = np.random.default_rng(k)
    du = 1.0 / (n * cell)
    at = np.repeat(np.arange(k), rng.integers(1, 40, k))[:k + skip]
    step = rng.uniform(-0.52 * n, 0.52 * n, (2, at.max() + 1))   # some runs fall off the grid
    u, v = ((step[q][at] * du).astype(np.float32) for q in range(2))
    vis = (rng.normal(size=k + skip) + 1j * rng.normal(size=k + skip)).astype(np.complex64)
    w = rng.uniform(0.2, 2.0, k + skip).astype(np.float32)
    wd = _dev(w)[skip:] if weighted else None
    g, ws = qc.image_grid(_dev(u)[skip:], _dev(v)[skip:], _dev(vis)[skip:], n, cell, weight=wd)
    u, v, vis = u[skip:], v[skip:], vis[skip:]
    w = w[skip:] if weighted else np.ones(k, np.float32)
    G_ref, W_ref = imaging.grid_nearest(u, v, vis, w, n, cell)
    mag, _ = imaging.grid_nearest(u, v, np.abs(vis), w, n, cell)
    cnt, _ = imaging.grid_nearest(u, v, np.ones(k), np.ones(k), n, cell)
    assert np.all(np.abs(g.cpu().numpy() - G_ref) <= (cnt.real + 2) * 2.0 ** -24 * 2 * mag.real)
    assert ws.item() == pytest.approx(W_ref, rel=1e-12)

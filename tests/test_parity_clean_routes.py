"""GPU parity of the ways a CLEAN launch can run: its workgroups together, alone
on the first one because the others were not there in time, alone because no
exchange area was free, and two launches in flight at once.  Components and
residual are bit-identical to the oracle each time, the count included."""

import numpy as np
import pytest

from oracle import imaging

pytestmark = pytest.mark.gpu


def _input(n, seed):
    rng = np.random.default_rng(seed)
    D = (rng.integers(-64, 65, (n, n)) / 64).astype(np.float32)
    P = (rng.integers(-16, 17, (n, n)) / 64).astype(np.float32)
    P[n // 2, n // 2] = 1.0
    return D, P


class _Launch:
    """One qc_image_clean on a stream of its own, not waited for."""

    def __init__(self, qc, D, P, gain, thr, iters):
        import torch
        self.qc, self.args, self.n, self.iters = qc, (gain, thr), D.shape[0], iters
        self.res, self.psf = torch.from_numpy(D.copy()).cuda(), torch.from_numpy(P).cuda()
        self.pix = torch.zeros(max(iters, 1), dtype=torch.int32, device="cuda")
        self.flux = torch.zeros(max(iters, 1), dtype=torch.float32, device="cuda")
        self.count = torch.full((1,), -7, dtype=torch.int32, device="cuda")
        self.stream = torch.cuda.Stream()
        self.ref = imaging.hogbom(D, P, gain, thr, iters)

    def go(self):
        st = self.qc.lib().qc_image_clean(self.res.data_ptr(), self.psf.data_ptr(), self.n, *self.args, self.iters,
                                          self.pix.data_ptr(), self.flux.data_ptr(), self.count.data_ptr(),
                                          self.stream.cuda_stream)
        assert st == 0

    def check(self):
        pix, flux, res = self.ref
        k = int(self.count.item())
        assert k == len(pix)
        assert np.array_equal(self.pix[:k].cpu().numpy(), pix)
        assert np.array_equal(self.flux[:k].cpu().numpy(), flux)
        assert np.array_equal(self.res.cpu().numpy(), res)


@pytest.fixture
def limits(qc):
    yield lambda areas, us: qc.lib().qc_image_clean_limits(areas, us)
    assert qc.lib().qc_image_clean_limits(-1, -1) == 0


@pytest.mark.parametrize("areas,gather_us", [(0, -1), (-1, 0), (-1, -1)])
@pytest.mark.parametrize("n,iters,thr", [(128, 20, 0.0), (128, 0, 0.0), (512, 9, 0.0), (512, 5, 9.0), (1024, 6, 0.0),
                                         (2048, 4, 0.0)])
def test_routes_agree(qc, limits, n, iters, thr, areas, gather_us):
    import torch
    one = _Launch(qc, *_input(n, n + iters), 0.3, thr, iters)
    torch.cuda.synchronize()
    assert limits(areas, gather_us) == 0
    one.go()
    torch.cuda.synchronize()
    one.check()


@pytest.mark.parametrize("areas,gather_us", [(-1, -1), (1, -1), (1, 0)])
def test_launches_in_flight(qc, limits, areas, gather_us):
    """Launches queued on four streams before any is waited for, twice over."""
    import torch
    made = [_Launch(qc, *_input(n, 3 * n + q), 0.2, 0.0, 25) for q, n in enumerate((512, 256, 512, 128))]
    again = [_Launch(qc, *_input(n, 5 * n + q), 0.2, 0.0, 25) for q, n in enumerate((128, 512, 256, 512))]
    for first, second in zip(made, again):
        second.stream = first.stream
    torch.cuda.synchronize()
    assert limits(areas, gather_us) == 0
    for one in made + again:
        one.go()
    torch.cuda.synchronize()
    for one in made + again:
        one.check()


@pytest.mark.parametrize("n", [64, 512, 8192])
def test_zero_at_the_last_pixel(qc, n):
    """The last pixel is a peak like any other, also where it is zero and the
    rest of the image is no number."""
    import torch
    D = np.full((n, n), np.nan, np.float32)
    D[-1, -1] = 0.0
    res, psf = torch.from_numpy(D).cuda(), torch.zeros((n, n), device="cuda")
    pix, flux = qc.image_clean(res, psf, 0.5, 0.0, 2)
    assert pix.cpu().numpy().tolist() == [n * n - 1] * 2
    assert flux.cpu().numpy().tolist() == [0.0, 0.0]


def test_limits_reject(qc):
    assert qc.lib().qc_image_clean_limits(17, 0) == -1
    assert qc.lib().qc_image_clean_limits(0, 1000001) == -1


@pytest.mark.parametrize("n", [64, 512])
def test_in_a_graph(qc, n):
    """A captured CLEAN claims and gives back an area on each replay; eager work and
    a CLEAN outside the graph run in between."""
    import torch
    one, other = (_Launch(qc, *_input(n, n + q), 0.3, 0.0, 12) for q in (1, 2))
    D, E = one.res.clone(), other.res.clone()
    one.go()                                     # first use outside the capture
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    one.stream.wait_stream(torch.cuda.current_stream())
    with torch.cuda.graph(graph, stream=one.stream):
        one.go()
    for _ in range(20):
        one.res.copy_(D)
        other.res.copy_(E)
        one.count.fill_(-7)
        torch.cuda.synchronize()
        graph.replay()
        other.go()
        torch.cuda.synchronize()
        one.check()
        other.check()

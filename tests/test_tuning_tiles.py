"""The fused F+X's tile lists: nothing that could be chosen is lost, and a shape
that stands twice is timed once."""

import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,n_ant,twice,count", [(4096, 4, (0, 6), 8), (4096, 2, (0, 4), 6), (1024, 8, (0, 1), 3)])
def test_shapes_that_stand_twice(qc, N, n_ant, twice, count):
    import torch
    x = torch.randint(-50, 51, (n_ant, 64 * N), dtype=torch.int8, device="cuda")
    assert qc.fx_tile_count(N, n_ant) == count
    try:
        best, ms = qc.fx_autotune(x, N, 4, 16, reps=1)
        assert ms[twice[0]] == ms[twice[1]] and best != twice[1]
        assert min(ms) > 0
    finally:
        qc.fx_set_tile(N, n_ant, 0)
        qc.fx_set_width(N, n_ant, 0)

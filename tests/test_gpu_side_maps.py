"""The stage kernels read periodic and open sides through an index map instead
of filled ghost layers, and directions of fewer cells than the halo is deep
from filled ones: both against the oracle, bit for bit, where the map can go
wrong (one, two, three and four cells across, mixed sides, a background)."""

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny", [(1, 24), (2, 24), (3, 17), (4, 9), (24, 1), (24, 2), (17, 3), (123, 4), (245, 11)])
@pytest.mark.parametrize("open_x,open_y", [(0, 0), (1, 0), (0, 1), (1, 1)])
@pytest.mark.parametrize("background", [False, True])
def test_side_maps_match_oracle(oracle_lib, nx, ny, open_x, open_y, background):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1710_06423_amd import Solver
    if (open_x and nx == 1) or (open_y and ny == 1):
        pytest.skip("a one-cell direction is periodic")
    print(f"case: {nx}x{ny} open {open_x}{open_y} background {background}", flush=True)
    prob = W.random_smooth(nx, ny, seed=nx + 31 * ny, bc=(open_x, open_x, open_y, open_y))
    if background:
        prob = W.split_background(prob, 0.4, 0.9, (0.1, -0.2))
    s = Solver.from_problem(prob)
    s.advance(4)
    got = s.read_fields().cpu().numpy()
    ora = oracle_lib.State(prob, form=oracle_lib.LOWSTORE)
    ora.run(4)
    assert np.array_equal(got, ora.stacked())
    assert s.diagnostics()["t"] == ora.t
    s.close()

"""The box kernel with four rows per block (FP64 with hyper-diffusion, as many
blocks as compute units or fewer), against the oracle, bit for bit, at the
edges of its 58 x 4 tile and of its range (256 blocks)."""

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny", [(3, 3), (57, 3), (58, 4), (59, 5), (64, 7), (116, 8), (117, 9), (232, 256), (233, 256)])
@pytest.mark.parametrize("open_x,open_y", [(0, 0), (1, 0), (0, 1), (1, 1)])
def test_four_row_boxes_match_oracle(oracle_lib, nx, ny, open_x, open_y):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1710_06423_amd import Solver
    prob = W.random_smooth(nx, ny, seed=nx + 31 * ny, bc=(open_x, open_x, open_y, open_y))
    print(f"case: {nx}x{ny} open {open_x}{open_y}", flush=True)
    s = Solver.from_problem(prob)
    s.advance(3)
    got = s.read_fields().cpu().numpy()
    ora = oracle_lib.State(prob, form=oracle_lib.LOWSTORE)
    ora.run(3)
    assert np.array_equal(got, ora.stacked())
    assert s.diagnostics()["t"] == ora.t
    s.close()

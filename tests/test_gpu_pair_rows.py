"""Two stages per launch with 24 and with 8 rows per block: the bits of one
stage per launch on both sides of the line between them."""

import pytest

import workloads as W

pytestmark = pytest.mark.gpu


# on 256 compute units: 24 rows (their only round against two of 8), 8 (two
# against two), 24 (two full ones against three), 8 in FP64 and 24 in FP32
@pytest.mark.parametrize("nx,ny", [(392, 600), (700, 500), (900, 697), (1501, 997)])
@pytest.mark.parametrize("precision", [0, 1])
def test_rows_keep_the_bits(nx, ny, precision):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1710_06423_amd import Solver
    print(f"case: {nx}x{ny} precision {precision}", flush=True)
    prob = W.random_smooth(nx, ny, seed=2, bc=(0, 0, 1, 1))
    a, b = (Solver.from_problem(prob, precision=precision, hd_on=False) for _ in range(2))
    b.set_launch(128, 33)
    a.advance(2)
    b.advance(2)
    assert torch.equal(a.read_fields(), b.read_fields())
    a.close()
    b.close()

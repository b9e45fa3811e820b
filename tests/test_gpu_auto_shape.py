"""The automatic launch shape (columns and rows per block) of small grids:
the same bits as a fixed shape, at sizes on both sides of its choices."""

import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny", [(58, 9), (59, 10), (64, 64), (123, 200), (300, 136), (1024, 64), (40, 1000), (1030, 1001)])
@pytest.mark.parametrize("precision,hd,background", [(0, True, False), (0, False, False), (0, True, True),
                                                     (1, True, False), (1, False, False)])
def test_automatic_shape_equals_fixed_shape(nx, ny, precision, hd, background):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1710_06423_amd import Solver
    prob = W.random_smooth(nx, ny, seed=nx + ny, bc=(1, 1, 0, 0))
    if background:
        prob = W.split_background(prob, 0.4, 0.9, (0.1, -0.2))
    out = []
    for shape in (None, (128, 33)):
        s = Solver.from_problem(prob, precision=precision, hd_on=hd)
        if shape:
            s.set_launch(*shape)
            assert s.get_launch() == shape
        print(f"case: {nx}x{ny} precision {precision} hd {hd} background {background} {s.get_launch()}", flush=True)
        s.advance(3)
        out.append(s.read_fields())
        s.close()
    assert torch.equal(out[0], out[1])


def test_rows_alone_take_the_default_width():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1710_06423_amd import Solver
    for precision, columns in ((0, 128), (1, 256)):
        s = Solver.from_problem(W.random_smooth(64, 64, seed=1), precision=precision)
        s.set_launch(0, 12)
        assert s.get_launch() == (columns, 12)
        s.close()

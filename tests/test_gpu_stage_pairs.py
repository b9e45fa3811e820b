"""Two stages per launch without hyper-diffusion: the bits of one stage per
launch (a launch shape set by hand takes those) at the edges of the 56-column
tile and its rows, with every kind of side, for even and odd numbers of steps,
gravity, an end time between the steps of a pair, and against the oracle."""

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


def _run(prob, precision, shape, calls, **kw):
    from paper_1710_06423_amd import Solver
    s = Solver.from_problem(prob, precision=precision, hd_on=False, **kw)
    if shape:
        s.set_launch(*shape)
    res = [s.advance(n, t_end) for n, t_end in calls]
    out = s.read_fields()
    d = s.diagnostics()
    s.close()
    return res, out, d


# one short of, at and past one tile and two; rows likewise; 7 cells across
# take one stage per launch in both; the last two have 24 rows per block
@pytest.mark.parametrize("nx,ny", [(8, 8), (7, 40), (55, 15), (56, 16), (57, 17), (58, 18), (112, 32), (113, 33),
                                   (60, 9), (300, 136), (950, 655), (952, 673)])
@pytest.mark.parametrize("open_x,open_y", [(0, 0), (1, 0), (0, 1), (1, 1)])
@pytest.mark.parametrize("precision", [0, 1])
def test_pairs_equal_single_stages(nx, ny, open_x, open_y, precision):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    prob = W.random_smooth(nx, ny, seed=nx + ny, bc=(open_x, open_x, open_y, open_y))
    prob.g = (0.1, -0.3)
    for calls in ([(4, 0.0)], [(3, 0.0)], [(2, 0.0), (1, 0.0), (2, 0.0)]):
        print(f"case: {nx}x{ny} open {open_x}{open_y} precision {precision} {calls}", flush=True)
        a, b = (_run(prob, precision, shape, calls) for shape in (None, (64, 33)))
        assert a[0] == b[0] and torch.equal(a[1], b[1])
        assert a[2] == b[2]


# the end time falls within the first, second, third and fourth step
@pytest.mark.parametrize("steps", [0.5, 1.5, 2.5, 3.0, 3.5])
def test_end_time_within_a_pair(steps):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    prob = W.random_smooth(70, 40, seed=3, bc=(0, 0, 1, 1))
    dt = _run(prob, 0, (64, 33), [(1, 0.0)])[2]["dt"]
    a, b = (_run(prob, 0, shape, [(6, steps * dt)]) for shape in (None, (64, 33)))
    assert a[0] == b[0] and torch.equal(a[1], b[1]) and a[2] == b[2]


@pytest.mark.parametrize("nx,ny", [(57, 17), (150, 70), (1009, 505)])
def test_pairs_match_oracle(oracle_lib, nx, ny):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    prob = W.random_smooth(nx, ny, seed=9, bc=(1, 1, 0, 0))
    res, out, d = _run(prob, 0, None, [(4, 0.0)])
    ora = oracle_lib.State(prob, form=oracle_lib.LOWSTORE, hd_on=False)
    ora.run(4)
    assert np.array_equal(out.cpu().numpy(), ora.stacked()) and d["t"] == ora.t

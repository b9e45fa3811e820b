"""The largest wave speed of a state is found wherever it is: one fast cell at
the first, middle and last lanes of waves and blocks and in blocks that share
an accumulator word, in the initial state and after a step, in 2-D and 3-D."""

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

# The speeds are a dozen roundings of the same operations here and there:
# 16 eps, where a missed cell would change the maximum by a factor of 20.
RTOL = 16 * 2.0 ** -52


def _speeds(f, gamma, nd):
    """|v_d| + c_f per direction, maximum over the cells (fields rho, m, e, B)."""
    rho, m, e, b = f[0], f[1:1 + nd], f[1 + nd], f[2 + nd:]
    v = m / rho
    b2 = (b * b).sum(0)
    p = (gamma - 1.0) * ((e - 0.5 * (m * v).sum(0)) - 0.5 * b2)
    c = np.sqrt((gamma * p + b2) / rho)
    return [float((np.abs(v[d]) + c).max()) for d in range(nd)]


@pytest.mark.parametrize("nx,ny", [(64, 48), (300, 9), (700, 1), (130, 260)])
@pytest.mark.parametrize("where", [(0.0, 0.0), (1.0, 1.0), (0.5, 0.5), (0.2, 0.9), (0.77, 0.31)])
def test_fast_cell_2d(nx, ny, where):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1710_06423_amd import Solver
    prob = W.random_smooth(nx, ny, seed=1, bc=(0, 0, 0, 0))
    f = {k: np.array(v) for k, v in prob.fields.items()}
    at = (round(where[1] * (ny - 1)), round(where[0] * (nx - 1)))
    f["rho"][at] /= 400.0
    f["mx"][at] /= 400.0
    f["my"][at] /= 400.0
    prob.fields.update(f)
    s = Solver.from_problem(prob, cfl=0.01)
    for step in range(2):
        d = s.diagnostics()
        got = s.read_fields().cpu().numpy()
        ref = _speeds(got, prob.gamma, 2)
        print(f"case: {nx}x{ny} cell {at} step {step}: {d['c_x']} {d['c_y']} {ref}", flush=True)
        assert abs(d["c_x"] - ref[0]) <= RTOL * ref[0] and abs(d["c_y"] - ref[1]) <= RTOL * ref[1]
        s.advance(1)
    s.close()


@pytest.mark.parametrize("hd", [True, False])
@pytest.mark.parametrize("where", [(0, 0, 0), (39, 17, 9), (31, 7, 4), (32, 8, 5)])
def test_fast_cell_3d(hd, where):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1710_06423_amd.sacx3 import Solver3
    prob = W.random_smooth_3d(40, 18, 10, seed=1)
    at = where[::-1]
    for n in ("rho", "mx", "my", "mz"):   # 1/400 of the density, the same velocity: 20 times the speed
        prob.fields[n] = np.array(prob.fields[n])
        prob.fields[n][at] /= 400.0
    s = Solver3.from_problem(prob, cfl=0.01, hd_on=hd)
    for step in range(2):
        d = s.diagnostics()
        ref = _speeds(s.read_fields().cpu().numpy(), prob.gamma, 3)
        print(f"case: 3-D cell {at} hd {hd} step {step}: {d['c']} {ref}", flush=True)
        assert all(abs(a - b) <= RTOL * b for a, b in zip(d["c"], ref))
        s.advance(1)
    s.close()

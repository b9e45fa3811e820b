"""A tube's whole steps in one launch each (pairs of steps of one call) against
the oracle and against single steps, which run stage by stage: lengths around
its blocks' 40 cells, and 232 from 10241 cells on, both kinds of ends, and calls that stop inside a pair."""

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


def _torch():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def _tube(n, bc, seed=3):
    return W.random_smooth(n, 1, seed=seed + n, bc=(bc[0], bc[1], 0, 0))


@pytest.mark.parametrize("n", [2, 3, 5, 23, 39, 40, 41, 80, 231, 232, 233, 464, 801, 10240, 10241, 10440])
@pytest.mark.parametrize("bc", [(0, 0), (1, 1)])
@pytest.mark.parametrize("hd", [True, False])
def test_tube_steps_match_oracle(oracle_lib, n, bc, hd):
    _torch()
    from paper_1710_06423_amd import Solver
    print(f"case: tube {n} bc {bc} hd {hd}", flush=True)
    prob = _tube(n, bc)
    s = Solver.from_problem(prob, hd_on=hd)
    s.advance(5)
    ora = oracle_lib.State(prob, form=oracle_lib.LOWSTORE, hd_on=hd)
    ora.run(5)
    assert np.array_equal(s.read_fields().cpu().numpy(), ora.stacked())
    assert s.diagnostics()["t"] == ora.t
    s.close()


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("gravity", [False, True])
def test_pairs_equal_single_steps(precision, gravity):
    torch = _torch()
    from paper_1710_06423_amd import Solver
    for n, bc in ((3, (0, 0)), (240, (1, 1)), (700, (0, 0)), (930, (1, 1))):
        print(f"case: tube {n} precision {precision} gravity {gravity}", flush=True)
        prob = _tube(n, bc)
        if gravity:
            prob = W.with_gravity(prob, (0.2, -0.3))
        a, b = Solver.from_problem(prob, precision=precision), Solver.from_problem(prob, precision=precision)
        a.advance(6)
        for _ in range(6):
            b.advance(1)
        assert torch.equal(a.read_fields(), b.read_fields())
        assert a.diagnostics() == b.diagnostics()
        a.close()
        b.close()


@pytest.mark.parametrize("stop", [0, 1, 2, 3])
def test_end_time_inside_a_pair(oracle_lib, stop):
    """t_end reached after `stop` full steps and one shortened one."""
    _torch()
    from paper_1710_06423_amd import Solver
    prob = W.brio_wu(300)
    ora = oracle_lib.State(prob, form=oracle_lib.LOWSTORE)
    ora.run(stop)
    t0 = ora.t
    ora.run(1)
    t_end = 0.5 * (t0 + ora.t)
    ref = oracle_lib.State(prob, form=oracle_lib.LOWSTORE)
    ref.run(stop)
    s = Solver.from_problem(prob)
    done, t = s.advance(10, t_end=t_end)
    print(f"case: stop {stop}: {done} steps, t = {t}", flush=True)
    assert done == stop + 1 and t == t_end
    one = Solver.from_problem(prob)
    for _ in range(stop + 1):
        one.advance(1, t_end=t_end)
    assert np.array_equal(s.read_fields().cpu().numpy(), one.read_fields().cpu().numpy())
    s.advance(3)
    one.advance(1); one.advance(1); one.advance(1)
    assert np.array_equal(s.read_fields().cpu().numpy(), one.read_fields().cpu().numpy())
    s.close()
    one.close()


def test_non_physical_inside_a_pair():
    """A state that turns non-physical stops a call wherever the step falls."""
    _torch()
    from paper_1710_06423_amd import Solver, sacx
    prob = W.brio_wu(200)
    a = Solver.from_problem(prob, hd_on=False)   # breaks down within a few steps
    b = Solver.from_problem(prob, hd_on=False)
    rc, done, t = a.advance_rc(40)
    total = 0
    while total < 40:
        rcb, n, tb = b.advance_rc(1)
        total += n
        if rcb != sacx.OK:
            break
    assert rc == rcb == sacx.ENONPHYS and done == total and t == tb
    assert np.array_equal(a.read_fields().cpu().numpy(), b.read_fields().cpu().numpy(), equal_nan=True)
    a.close()
    b.close()

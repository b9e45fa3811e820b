"""The domain's launches over all subdomains: rebuilt after a change of a
subdomain's settings, replaced by per-subdomain launches under capture and for
narrow periodic directions; always the undivided run's bits."""

import pytest

import workloads as W

pytestmark = pytest.mark.gpu


def _torch():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


@pytest.mark.parametrize("precision,hd", [(0, True), (0, False), (1, True), (1, False)])
@pytest.mark.parametrize("shape,xc,yc,bc", [
    ((131, 77), [0, 64, 131], [0, 3, 77], (0, 0, 0, 0)),
    ((131, 77), [0, 131], [0, 30, 77], (1, 1, 0, 0)),
    ((60, 90), [0, 20, 40, 60], [0, 90], (0, 0, 1, 1)),
    ((90, 2), [0, 40, 90], [0, 2], (0, 0, 0, 0)),
])
def test_rebuilt_tables_keep_the_bits(precision, hd, shape, xc, yc, bc):
    torch = _torch()
    from paper_1710_06423_amd import DecomposedSolver, Solver
    prob = W.random_smooth(*shape, seed=5, bc=bc)
    print(f"case: {shape} cuts {xc} {yc} bc {bc} precision {precision} hd {hd}", flush=True)
    one = Solver.from_problem(prob, precision=precision, hd_on=hd)
    d = DecomposedSolver(prob, xc, yc, precision=precision, hd_on=hd)
    last = d.subs[-1][-1]
    for change in (lambda: None, lambda: last.set_launch(64, 5), lambda: last.set_column_split(False),
                   lambda: d.subs[0][0].set_launch(256, 0)):
        change()
        d.advance(2)
        one.advance(2)
        assert torch.equal(d.read_fields(), one.read_fields())
    assert d.diagnostics()[0][0]["t"] == one.diagnostics()["t"]
    d.close()
    one.close()


def test_eager_calls_between_replays():
    """A captured piece of a domain keeps its own launches: eager calls with
    other settings between its replays do not change what it does."""
    torch = _torch()
    from paper_1710_06423_amd import DecomposedSolver, Solver
    prob = W.orszag_tang(96, ny=70)
    print("case: domain graph between eager calls", flush=True)
    one = Solver.from_problem(prob)
    d = DecomposedSolver(prob, [0, 50, 96], [0, 30, 70], stream=torch.cuda.Stream())
    d.advance(1)
    g = d.graph(2)
    for rows in (0, 7, 30):
        if rows:
            d.subs[0][1].set_launch(64, rows)
        g.replay()
        d.advance(1)
    torch.cuda.synchronize()
    one.advance(10)
    assert torch.equal(d.read_fields(), one.read_fields())
    d.close()
    one.close()


@pytest.mark.parametrize("precision,shape,xc,yc", [
    (0, (4003, 4001), [0, 2002, 4003], [0, 2000, 4001]),   # stages launched by subdomain
    (0, (4003, 3900), [0, 2002, 4003], [0, 1950, 3900]),   # from one list, several rounds of blocks
    (1, (5800, 2900), [0, 2900, 5800], [0, 2900]),
])
def test_large_subdomains_keep_the_bits(precision, shape, xc, yc):
    torch = _torch()
    from paper_1710_06423_amd import DecomposedSolver, Solver
    prob = W.orszag_tang(shape[0], ny=shape[1])
    print(f"case: {shape} cuts {xc} {yc} precision {precision}", flush=True)
    one = Solver.from_problem(prob, precision=precision)
    d = DecomposedSolver(prob, xc, yc, precision=precision)
    d.advance(3)
    one.advance(3)
    assert torch.equal(d.read_fields(), one.read_fields())
    assert d.diagnostics()[0][0]["t"] == one.diagnostics()["t"]
    d.close()
    one.close()

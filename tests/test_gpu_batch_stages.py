"""Batches by stage launches (the default) and by the persistent launch: the
same bits, with instances of one, two and few rows and any tile shape."""

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("tiles", [None, (64, 1), (256, 300)])
def test_stage_launches_equal_the_persistent_launch(monkeypatch, precision, tiles):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1710_06423_amd import Batch, Solver
    probs = [W.orszag_tang(131, ny=2), W.brio_wu(59), W.random_smooth(3, 40, seed=1), W.brio_wu(700),
             W.random_smooth(130, 65, seed=2, bc=(1, 1, 0, 0)), W.orszag_tang(64, ny=3)]
    print(f"case: precision {precision} tiles {tiles}", flush=True)
    out = []
    for bound in (None, "1048576"):
        if bound is None:
            monkeypatch.delenv("SACX_BATCH_SPIN_LIMIT", raising=False)
        else:
            monkeypatch.setenv("SACX_BATCH_SPIN_LIMIT", bound)
        b = Batch(probs, precision=precision)
        if tiles:
            b.set_tiles(tiles[0], [tiles[1]] * len(probs))
        b.advance(3)
        b.advance(4)
        out.append([b[i].read_fields().cpu().numpy() for i in range(len(probs))])
        b.close()
    for i, p in enumerate(probs):
        s = Solver.from_problem(p, precision=precision)
        s.advance(7)
        assert np.array_equal(out[0][i], out[1][i]), i
        assert np.array_equal(out[0][i], s.read_fields().cpu().numpy()), i
        s.close()


@pytest.mark.parametrize("precision,sizes", [
    (0, [(2600, 2400), (2500, 2600), (2400, 2500), (2700, 2500)]),   # one round of strips longer than 256 rows
    (1, [(3000, 2900), (2900, 3000), (3000, 3000), (2800, 3000)]),
])
def test_large_instances_equal_single_runs(precision, sizes):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1710_06423_amd import Batch, Solver
    print(f"case: {sizes} precision {precision}", flush=True)
    probs = [W.orszag_tang(nx, ny=ny) for nx, ny in sizes]
    b = Batch(probs, precision=precision)
    b.advance(2)
    for i, p in enumerate(probs):
        s = Solver.from_problem(p, precision=precision)
        s.advance(2)
        assert torch.equal(b[i].read_fields(), s.read_fields())
        s.close()
    b.close()

"""Instances of two rows: their ghost rows take one launch per stage for all
of them."""

import ctypes

import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", [0, 1])
def test_launches_do_not_grow_with_the_instances(precision):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1710_06423_amd import Batch, Solver, sacx
    lib = sacx.load_library()
    probs = [W.orszag_tang(32 + 7 * i, ny=2) for i in range(40)] + [W.brio_wu(90), W.orszag_tang(48, ny=33),
                                                                  W.random_smooth(3000, 2, seed=1)]
    print(f"case: {len(probs)} instances precision {precision}", flush=True)
    b = Batch(probs, precision=precision, stream=torch.cuda.Stream())
    b.advance(1)
    steps = 3
    g = torch.cuda.CUDAGraph(keep_graph=True)
    torch.cuda.synchronize()
    with torch.cuda.graph(g, stream=b.stream, capture_error_mode="thread_local"):
        b.advance(steps, sync=False)
    n = ctypes.c_size_t(0)
    assert lib.hipGraphGetNodes(ctypes.c_void_p(g.raw_cuda_graph()), None, ctypes.byref(n)) == 0
    print(f"nodes: {n.value}", flush=True)
    # per step the scalars, then per stage the ghost rows and the tiles; a flag cleared and the last scalars
    assert n.value <= 9 * steps + 2
    b.advance(2)
    for i, p in enumerate(probs):
        s = Solver.from_problem(p, precision=precision)
        s.advance(3)
        assert torch.equal(b[i].read_fields(), s.read_fields()), i
        s.close()
    b.close()

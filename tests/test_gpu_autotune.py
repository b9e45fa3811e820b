"""Tuning never leaves a program slower than it was untuned, and a set shape
can be taken back."""

import json

import pytest

import workloads as W

pytestmark = pytest.mark.gpu

# tuned and untuned runs are the same launches where nothing beats the
# automatic ones; short timings scatter by a few percent
SLACK = 1.15


def _torch():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def _ms(torch, advance, stream, n):
    best = []
    for _ in range(5):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        torch.cuda.synchronize()
        a.record(stream)
        advance(n)
        b.record(stream)
        torch.cuda.synchronize()
        best.append(a.elapsed_time(b) / n)
    return min(best)


@pytest.mark.parametrize("shape,precision,hd", [((300, 136), 0, True), ((512, 512), 0, False), ((400, 300), 1, True),
                                               ((800, 1), 0, True)])
def test_tuned_solver_is_no_slower(shape, precision, hd):
    torch = _torch()
    from paper_1710_06423_amd import Solver
    from paper_1710_06423_amd.autotune import tune_solver
    print(f"case: {shape} precision {precision} hd {hd}", flush=True)
    prob = W.random_smooth(*shape, seed=1) if shape[1] > 1 else W.brio_wu(shape[0])
    plain, tuned = (Solver.from_problem(prob, precision=precision, hd_on=hd) for _ in range(2))
    t, r = tune_solver(tuned)
    assert t in (64, 128, 256) and r in (32, 64, 128, 256)
    ms = [_ms(torch, lambda n, s=s: s.advance(n, sync=False), s.stream, 40) for s in (plain, tuned)]
    print(f"[autotune] untuned {ms[0]:.4f} tuned {ms[1]:.4f} ms/step", flush=True)
    assert ms[1] <= SLACK * ms[0]
    plain.close()
    tuned.close()


@pytest.mark.parametrize("precision", [0, 1])
def test_tuned_batch_is_no_slower(precision):
    torch = _torch()
    from paper_1710_06423_amd import Batch
    from paper_1710_06423_amd.autotune import tune_batch
    probs = W.batch_instances(seed=2, n_bw=8, n_ot=8)
    print(f"case: {len(probs)} instances precision {precision}", flush=True)
    plain, tuned = Batch(probs, precision=precision), Batch(probs, precision=precision)
    t, r, trials = tune_batch(tuned, use_cache=False)
    assert t and r and trials[0][:2] == (0, 0) and len(trials) == 9
    ms = [_ms(torch, lambda n, b=b: b.advance(n, sync=False), b.stream, 10) for b in (plain, tuned)]
    print(f"[autotune] untuned {ms[0]:.4f} tuned {ms[1]:.4f} ms/step, tiles {tuned.tiles}", flush=True)
    assert ms[1] <= SLACK * ms[0]
    plain.close()
    tuned.close()


def test_back_to_the_automatic_launches():
    torch = _torch()
    from paper_1710_06423_amd import Batch, Solver
    print("case: automatic again", flush=True)
    for prob in (W.orszag_tang(300, ny=136), W.orszag_tang(2100, ny=1900)):
        a, b = Solver.from_problem(prob), Solver.from_problem(prob)
        chosen = b.get_launch()
        for shape in ((64, 7), (0, 9), (256, 0)):
            b.set_launch(*shape)
            assert b.get_launch() != chosen
            b.advance(1)
            b.set_launch_auto()
            assert b.get_launch() == chosen
            b.advance(1)
            a.advance(2)
            assert torch.equal(a.read_fields(), b.read_fields())
        a.close()
        b.close()
    probs = [W.orszag_tang(200, ny=90), W.brio_wu(300)]
    a, b = Batch(probs), Batch(probs)
    b.set_tiles(64, [5, 5])
    assert b.tiles
    b.advance(1)
    b.set_tiles_auto()
    assert b.tiles is None
    b.advance(2)
    a.advance(3)
    for i in range(2):
        assert torch.equal(a[i].read_fields(), b[i].read_fields())
    a.close()
    b.close()


def test_cached_shapes_of_another_library_are_not_taken_over(monkeypatch, tmp_path):
    _torch()
    from paper_1710_06423_amd import Batch, autotune
    print("case: tuner cache", flush=True)
    monkeypatch.setattr(autotune, "CACHE", str(tmp_path / "autotune.json"))
    probs = [W.orszag_tang(200, ny=90), W.brio_wu(300)]
    b = Batch(probs)
    (tmp_path / "autotune.json").write_text(json.dumps({autotune.batch_signature(b): {"threads": 64, "rows2d": 1}}))
    t, r, trials = autotune.tune_batch(b, threads=(128,), rows2d=(16, 32))
    assert len(trials) == 3
    kept = b.tiles
    b.set_tiles(64, [1, 1])
    assert autotune.tune_batch(b, threads=(128,), rows2d=(16, 32)) == (t, r, [])
    assert b.tiles == kept
    b.close()

"""Profiling a domain's subdomains: each gets its share of the launches over
all of them."""

import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,xc,yc,steps", [
    ((300, 200), [0, 150, 300], [0, 120, 200], 3),
    ((4004, 4002), [0, 2002, 4004], [0, 2001, 4002], 2),   # stages launched by subdomain
])
def test_every_subdomain_has_its_times(shape, xc, yc, steps):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1710_06423_amd import DecomposedSolver
    print(f"case: {shape} cuts {xc} {yc}", flush=True)
    d = DecomposedSolver(W.orszag_tang(shape[0], ny=shape[1]), xc, yc)
    subs = [s for row in d.subs for s in row]
    d.advance(1)
    for chosen in (subs, subs[-1:]):
        for s in chosen:
            s.profile_enable(True)
        d.advance(steps)
        for s in chosen:
            p = s.profile_read()
            assert p["n_stage"] == [steps] * 4 and all(ms > 0 for ms in p["ms_stage"])
            assert p["n_halo"] > 0 and p["ms_halo"] > 0 and p["n_scalar"] > 0 and p["ms_scalar"] > 0
        for s in subs:
            s.profile_enable(False)
    # the shares of all subdomains add up to the launches' time
    torch.cuda.synchronize()
    for s in subs:
        s.profile_enable(True)
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    with torch.cuda.stream(d.stream):
        a.record()
        d.advance(steps)
        b.record()
    torch.cuda.synchronize()
    total = sum(sum(p["ms_stage"]) + p["ms_halo"] + p["ms_scalar"] for p in (s.profile_read() for s in subs))
    assert total <= a.elapsed_time(b)
    d.close()

"""Fields left out of a read are zero also where freed memory held other
values; with every field asked for, every element is the state's."""

import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mask", [0x3F, 0x15, 0x01, 0x00])
@pytest.mark.parametrize("dtype", ["float64", "float32"])
def test_mask_2d(mask, dtype):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1710_06423_amd import Solver
    prob = W.random_smooth(37, 11, seed=1)
    s = Solver.from_problem(prob)
    dt = getattr(torch, dtype)
    junk = torch.full((6, 11, 37), float("nan"), dtype=dt, device="cuda")
    del junk
    got = s.read_fields(dtype=dt, mask=mask)
    for k, name in enumerate(("rho", "mx", "my", "e", "bx", "by")):
        ref = torch.as_tensor(prob.fields[name]).to(dt).cuda() if mask >> k & 1 else torch.zeros_like(got[k])
        assert torch.equal(got[k], ref), (k, mask)
    s.close()


@pytest.mark.parametrize("mask", [0xFF, 0xA1, 0x00])
def test_mask_3d(mask):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1710_06423_amd.sacx3 import Solver3
    prob = W.random_smooth_3d(13, 7, 5, seed=1)
    s = Solver3.from_problem(prob)
    junk = torch.full((8, 5, 7, 13), float("nan"), dtype=torch.float64, device="cuda")
    del junk
    got = s.read_fields(mask=mask)
    for k, name in enumerate(("rho", "mx", "my", "mz", "e", "bx", "by", "bz")):
        ref = torch.as_tensor(prob.fields[name]).cuda() if mask >> k & 1 else torch.zeros_like(got[k])
        assert torch.equal(got[k], ref), (k, mask)
    s.close()

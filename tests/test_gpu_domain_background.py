"""A domain of one subdomain may carry a background (no side of it is an
exchange side): it steps as the context does alone."""

import ctypes

import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("hd", [True, False])
@pytest.mark.parametrize("shape", [(60, 70), (131, 3), (700, 500)])
def test_single_subdomain_keeps_its_background(precision, hd, shape):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1710_06423_amd import Solver, sacx
    lib = sacx.load_library()
    prob = W.stratified_atmosphere(*shape)
    print(f"case: {shape} precision {precision} hd {hd}", flush=True)
    one = Solver.from_problem(prob, precision=precision, hd_on=hd)
    sub = Solver.from_problem(prob, precision=precision, hd_on=hd)
    subs = (ctypes.c_void_p * 1)(sub.ctx.value)
    need = ctypes.c_size_t(0)
    assert lib.sacx_domain_buffer_size(1, 1, subs, ctypes.byref(need)) == sacx.OK
    buf = torch.empty(need.value + 256, dtype=torch.uint8, device="cuda")
    base = buf.data_ptr() + (-buf.data_ptr()) % 256
    d = ctypes.c_void_p(None)
    assert lib.sacx_domain_create(1, 1, subs, ctypes.c_void_p(base), need.value, ctypes.byref(d)) == sacx.OK
    for _ in range(2):
        assert lib.sacx_domain_advance(d, 3) == sacx.OK
        one.advance(3)
        assert torch.equal(sub.read_fields(), one.read_fields())
    assert sub.diagnostics()["t"] == one.diagnostics()["t"]
    assert lib.sacx_domain_destroy(d) == sacx.OK
    sub.close()
    one.close()

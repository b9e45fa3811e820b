"""sacx_stage runs on the state whose ghost cells the caller completed,
whatever the kind of the side they lie beyond; the state that sacx_init_state
leaves has its ghost cells filled."""

import ctypes

import pytest

import workloads as W

pytestmark = pytest.mark.gpu
PERIODIC, OPEN, EXCHANGE = 0, 1, 2


def _torch():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def _sub(torch, prob, i0, i1, j0, j1, bc, precision, hd):
    from paper_1710_06423_amd import Solver, sacx
    dx, dy = (prob.x1 - prob.x0) / prob.nx, (prob.y1 - prob.y0) / prob.ny
    g = sacx.make_grid(i1 - i0, j1 - j0, prob.x0 + i0 * dx, prob.x0 + i1 * dx, prob.y0 + j0 * dy, prob.y0 + j1 * dy,
                       precision, False)
    s = Solver(g, sacx.make_params(prob.gamma, 0.3, hd, True), bc)
    s.set_spacing(dx, dy)
    s.init_state(torch.stack([torch.from_numpy(prob.fields[k][j0:j1, i0:i1].copy()) for k in W.FIELDS]).cuda())
    return s


def _hand_over(subs, side):
    """One direction: every subdomain packs both its strips, then unpacks those
    that face it."""
    py, px = len(subs), len(subs[0])
    buf = {}
    for b in range(py):
        for a in range(px):
            for k in (side, side + 1):
                buf[b, a, k] = subs[b][a].halo_buffer(k)
                subs[b][a].halo_pack(k, buf[b, a, k])
    for b in range(py):
        for a in range(px):
            lo = ((a - 1) % px, b) if side == 0 else (a, (b - 1) % py)
            hi = ((a + 1) % px, b) if side == 0 else (a, (b + 1) % py)
            subs[b][a].halo_unpack(side, buf[lo[1], lo[0], side + 1])
            subs[b][a].halo_unpack(side + 1, buf[hi[1], hi[0], side])


@pytest.mark.parametrize("kind", [PERIODIC, OPEN])
@pytest.mark.parametrize("precision,hd", [(0, True), (0, False), (1, True), (1, False)])
@pytest.mark.parametrize("shape,xc,yc", [
    ((131, 77), [0, 64, 131], [0, 30, 77]),
    ((40, 900), [0, 3, 40], [0, 900]),
])
def test_strips_on_sides_of_any_kind(kind, precision, hd, shape, xc, yc):
    """A periodic domain cut into pieces whose sides are all `kind`: the
    strips that the caller unpacks are what the stages read."""
    torch = _torch()
    from paper_1710_06423_amd import Solver
    prob = W.random_smooth(*shape, seed=3)
    print(f"case: {shape} cuts {xc} {yc} kind {kind} precision {precision} hd {hd}", flush=True)
    one = Solver.from_problem(prob, precision=precision, hd_on=hd)
    subs = [[_sub(torch, prob, xc[a], xc[a + 1], yc[b], yc[b + 1], (kind,) * 4, precision, hd)
             for a in range(len(xc) - 1)] for b in range(len(yc) - 1)]
    flat = [s for row in subs for s in row]
    for _ in range(3):
        speeds = [s.wave_speeds() for s in flat]
        c = tuple(max(v[d] for v in speeds) for d in range(2))
        for _stage in range(4):
            _hand_over(subs, 0)
            _hand_over(subs, 2)
            for s in flat:
                s.stage(c)
    one.advance(3)
    ref = one.read_fields()
    for b, row in enumerate(subs):
        for a, s in enumerate(row):
            assert torch.equal(s.read_fields(), ref[:, yc[b]:yc[b + 1], xc[a]:xc[a + 1]]), (a, b)
    for s in flat + [one]:
        s.close()


@pytest.mark.parametrize("bc", [(0, 0, 0, 0), (1, 1, 0, 0), (0, 0, 1, 1), (1, 1, 1, 1)])
@pytest.mark.parametrize("shape", [(60, 44), (300, 2), (2, 50), (3, 4), (5, 3), (257, 9)])
def test_a_loaded_state_has_its_ghosts(bc, shape):
    """Stage 1 and the strips' corners right after the state is loaded, the
    second time over steps taken before, without a fill by the caller."""
    torch = _torch()
    from paper_1710_06423_amd import Solver
    prob = W.random_smooth(*shape, seed=4, bc=bc)
    print(f"case: {shape} bc {bc}", flush=True)
    a, b = Solver.from_problem(prob), Solver.from_problem(prob)
    a.advance(2)
    for load in (False, True):
        if load:   # a state loaded again after steps
            f = torch.stack([torch.from_numpy(prob.fields[k].copy()) for k in W.FIELDS]).cuda()
            a.init_state(f)
            b.init_state(f)
            a.advance(2)
        if shape[1] >= 3:
            strip = b.halo_buffer(2)
            b.halo_pack(2, strip)
            nx = shape[0]
            got = strip.view(torch.float64).reshape(6, 3, nx + 6)
            i = torch.arange(-3, nx + 3, device=got.device)
            i = i % nx if bc[0] == PERIODIC else i.clamp(0, nx - 1)
            assert torch.equal(got, b.read_fields()[:, :3][:, :, i])
        for _step in range(2):
            for st in range(4):
                if st or _step:
                    b.fill_boundaries(0)
                    b.fill_boundaries(1)
                b.stage(None)
        assert torch.equal(a.read_fields(), b.read_fields())
    a.close()
    b.close()


@pytest.mark.parametrize("hd", [True, False])
def test_background_ghosts_follow_the_boundaries(hd):
    torch = _torch()
    from paper_1710_06423_amd import Solver
    prob = W.stratified_atmosphere(90, 70, b_b=(0.3, 0.2))
    print(f"case: background, hd {hd}", flush=True)
    a, b = Solver.from_problem(prob, hd_on=hd), Solver.from_problem(prob, hd_on=hd)
    for bc in ((0, 0, 1, 1), (1, 1, 1, 1), (0, 0, 0, 0)):
        a.set_boundaries(bc)
        b.set_boundaries(bc)
        a.advance(2)
        for _ in range(8):
            b.fill_boundaries(0)
            b.fill_boundaries(1)
            b.stage(None)
        assert torch.equal(a.read_fields(), b.read_fields()), bc
    a.close()
    b.close()


@pytest.mark.parametrize("precision,hd", [(0, True), (0, False), (1, True)])
@pytest.mark.parametrize("kinds", [((PERIODIC, PERIODIC), (OPEN, OPEN)), ((OPEN, OPEN), (PERIODIC, PERIODIC)),
                                   ((EXCHANGE, EXCHANGE), (OPEN, OPEN))])
def test_neighbours_of_other_kinds(precision, hd, kinds):
    """Two subdomains one above the other whose x sides differ in kind: the
    corners travel with the y strips, in the domain object as in the stage-level
    calls."""
    torch = _torch()
    from paper_1710_06423_amd import sacx
    lib = sacx.load_library()
    prob = W.random_smooth(70, 60, seed=6)
    print(f"case: kinds {kinds} precision {precision} hd {hd}", flush=True)

    def pair():
        return [[_sub(torch, prob, 0, 70, j0, j1, k + (EXCHANGE, EXCHANGE), precision, hd)]
                for (j0, j1), k in zip(((0, 25), (25, 60)), kinds)]

    ours, theirs = pair(), pair()
    subs = (ctypes.c_void_p * 2)(*[r[0].ctx.value for r in theirs])
    need = ctypes.c_size_t(0)
    assert lib.sacx_domain_buffer_size(1, 2, subs, ctypes.byref(need)) == sacx.OK
    buf = torch.empty(need.value + 256, dtype=torch.uint8, device="cuda")
    base = buf.data_ptr() + (-buf.data_ptr()) % 256
    d = ctypes.c_void_p(None)
    assert lib.sacx_domain_create(1, 2, subs, ctypes.c_void_p(base), need.value, ctypes.byref(d)) == sacx.OK
    for _ in range(2):
        assert lib.sacx_domain_advance(d, 2) == sacx.OK
        for _step in range(2):
            speeds = [r[0].wave_speeds() for r in ours]
            c = tuple(max(v[k] for v in speeds) for k in range(2))
            for _stage in range(4):
                for r, k in zip(ours, kinds):
                    r[0].fill_boundaries(0)
                    if k[0] == EXCHANGE:   # its own neighbour across x
                        lo, hi = r[0].halo_buffer(0), r[0].halo_buffer(1)
                        r[0].halo_pack(0, lo)
                        r[0].halo_pack(1, hi)
                        r[0].halo_unpack(0, hi)
                        r[0].halo_unpack(1, lo)
                _hand_over(ours, 2)
                for r in ours:
                    r[0].stage(c)
        for r, q in zip(ours, theirs):
            assert torch.equal(r[0].read_fields(), q[0].read_fields())
    assert lib.sacx_domain_destroy(d) == sacx.OK
    for r in ours + theirs:
        r[0].close()


@pytest.mark.parametrize("kind,shape", [("orszag_tang", (60, 44)), ("brio_wu", (90, 1)), ("brio_wu", (50, 7)),
                                        ("brio_wu", (1, 70))])
@pytest.mark.parametrize("precision", [0, 1])
def test_a_generated_state_has_its_ghosts(kind, shape, precision):
    torch = _torch()
    from paper_1710_06423_amd import Solver, sacx
    print(f"case: {kind} {shape} precision {precision}", flush=True)
    which = sacx.PROBLEM_ORSZAG_TANG if kind == "orszag_tang" else sacx.PROBLEM_BRIO_WU
    runs = []
    for by_stage in (False, True):
        s = Solver(sacx.make_grid(*shape, 0.0, 1.0, 0.0, 1.0, precision, False), sacx.make_params(2.0))
        s.init_problem(which)
        if by_stage:
            for st in range(4):
                if st:
                    s.fill_boundaries(0)
                    s.fill_boundaries(1)
                s.stage(None)
        else:
            s.advance(1)
        runs.append(s.read_fields())
        s.close()
    assert torch.equal(*runs)


@pytest.mark.parametrize("kind", [PERIODIC, OPEN])
def test_a_captured_step_keeps_the_callers_ghosts(kind):
    """A step captured as the first stage-level calls, the strips of its later
    stages handed over inside, those of its first stage by the caller between
    the replays; on open sides that is not what a fill would put there.  On
    periodic ones the first replay reads the loaded state's own ghost cells."""
    torch = _torch()
    from paper_1710_06423_amd import Solver
    from paper_1710_06423_amd.sacx import StepGraph
    print(f"case: captured step, sides {kind}", flush=True)
    prob = W.random_smooth(60, 44, seed=8)
    one = Solver.from_problem(prob)
    s = Solver.from_problem(prob, stream=torch.cuda.Stream())
    if kind == OPEN:
        s.set_boundaries((OPEN,) * 4)
    strips = [s.halo_buffer(k) for k in range(4)]
    torch.cuda.synchronize()

    def hand_over():
        for side in (0, 2):
            s.halo_pack(side, strips[side])
            s.halo_pack(side + 1, strips[side + 1])
            s.halo_unpack(side, strips[side + 1])
            s.halo_unpack(side + 1, strips[side])

    def step():
        s.stage(None)
        for _ in range(3):
            hand_over()
            s.stage(None)

    g = StepGraph(step, s.stream)
    for k in range(4):
        if k or kind == OPEN:
            with torch.cuda.stream(s.stream):
                hand_over()
        g.replay()
        torch.cuda.synchronize()
        one.advance(1)
        assert torch.equal(s.read_fields(), one.read_fields()), k
    # a state loaded again is filled again
    f = torch.stack([torch.from_numpy(prob.fields[k].copy()) for k in W.FIELDS]).cuda()
    one.init_state(f)
    s.init_state(f)
    if kind == OPEN:
        with torch.cuda.stream(s.stream):
            hand_over()
    g.replay()
    torch.cuda.synchronize()
    one.advance(1)
    assert torch.equal(s.read_fields(), one.read_fields())
    s.close()
    one.close()

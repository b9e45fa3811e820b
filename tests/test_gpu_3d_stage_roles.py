"""GPU parity of the 3-D stage's two-role kernel (the columns' states and
ideal terms in one half of a block's waves, the face fluxes in the other) at
the edges of its 32 x 8 tile and of a block's strip of planes, bit for bit
against the 3-D oracle's low-storage form."""

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


# tiles: one column short, full, one over, one cell; strips: one plane, two
# (each parity of the first plane), a remainder, the automatic choice; sides
# of 1, 2 (periodic: filled ghost layers) and 3 cells (read in place)
@pytest.mark.parametrize("nx,ny,nz,planes,cross", [
    (31, 7, 5, 1, True),
    (32, 8, 6, 2, True),
    (33, 9, 7, 3, True),
    (1, 17, 11, 4, True),
    (65, 1, 9, 0, False),
    (64, 16, 1, 0, True),
    (3, 24, 2, 1, False),
    (4, 3, 5, 2, True),
    (2, 9, 3, 0, True),
])
@pytest.mark.parametrize("opened", [False, True])
def test_tile_and_strip_edges_bit_exact(nx, ny, nz, planes, cross, opened):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from oracle import oracle3d as O3
    from paper_1710_06423_amd.sacx3 import Solver3
    O3.build(force=False)
    bc = sum(((int(opened and n > 1),) * 2 for n in (nx, ny, nz)), ())
    prob = W.random_smooth_3d(nx, ny, nz, seed=5, bc=bc)
    print(f"case: {nx}x{ny}x{nz} planes={planes} cross={cross} bc={bc}", flush=True)
    s = Solver3.from_problem(prob, hd_cross_on=cross)
    if planes:
        s.set_launch(planes)
    done, t = s.advance(3)
    got = s.read_fields().cpu().numpy()
    ref = O3.State3(prob, form=O3.LOWSTORE, hd_cross_on=cross)
    ref.run(3)
    assert done == 3 and t == ref.t
    assert np.array_equal(got, ref.f)
    s.close()

"""Weight gradients of the network at the image heights where the row ring of
the gradient kernel can go wrong (fewer rows than the ring holds, one row per
block, ragged groups of rows), against the reference network."""

import numpy as np
import pytest

import workloads as W
from oracle import cnn

pytestmark = pytest.mark.gpu

# both sides round to BF16 at the same points; FP32 sums differ by about 1e-6,
# a rounding that falls on the other side of a boundary by one BF16 ulp of one
# value: relative 1e-3 over a layer's gradient
GRAD_REL = 1e-3


@pytest.mark.parametrize("shape", [(1, 1, 32), (1, 2, 32), (2, 3, 64), (1, 4, 96), (3, 5, 32), (4, 130, 128)])
def test_gradients_at_few_and_ragged_rows(shape):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1710_06423_amd import sacx as sx
    from paper_1710_06423_amd.surrogate import Network
    n, h, w = shape
    print(f"case: gradients {shape}", flush=True)
    p, x, t = W.cnn_case(n, h, w, seed=11 * h + w)
    p = {k: v.astype(np.float32).astype(np.float64) for k, v in p.items()}
    net = Network(torch.tensor(cnn.flatten(p), dtype=torch.float32))
    img = torch.zeros((n, h, w, 8), dtype=torch.float32)
    img[..., :6] = torch.from_numpy(x).permute(0, 2, 3, 1).to(torch.float32)
    img = img.to(torch.bfloat16)
    xr = img[..., :6].to(torch.float64).permute(0, 3, 1, 2).contiguous().numpy()
    target = t.astype(np.float32)
    loss = net.loss_of(img.cuda().contiguous(), torch.from_numpy(target).cuda())
    loss_ref, g_ref = cnn.batch_loss_and_grads(p, list(xr), list(target.astype(np.float64)), bf16=True)
    assert abs(loss - loss_ref) <= 1e-5 * loss_ref
    g, gr, o = net.grad.cpu().numpy().astype(np.float64), cnn.flatten(g_ref), 0
    for l, (ci, co) in enumerate(cnn.LAYERS):
        for size in (co * ci * 9, co):
            a, r = g[o:o + size], gr[o:o + size]
            assert np.linalg.norm(a - r) <= GRAD_REL * np.linalg.norm(r), (l, size)
            o += size

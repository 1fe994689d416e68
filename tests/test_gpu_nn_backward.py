"""Network gradients at the edges of the backward kernels' bricks (16 x 4 x 8 voxels).

The reference is the FP64 network oracle with bfloat16 rounding where the GPU pipeline stores
bfloat16; what remains is FP32 accumulation and rare rounding flips. A flip changes one masked
gradient or activation by 2^-8 of itself; a parameter block sums at least 16 voxels' worth of such
terms, so a block's relative error stays under a few 2^-8: 3e-2, and its direction within 0.999.
"""
import numpy as np
import pytest

from oracle import nn

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a HIP GPU")]

import paper_1112_3507_amd as hp  # noqa: E402


# smallest grid; bricks cut in every axis at each level; more bricks than one in z with a remainder;
# whole bricks
@pytest.mark.parametrize("n", [(4, 4, 4), (20, 12, 12), (36, 8, 20), (12, 20, 28), (32, 8, 16)])
def test_gradient_at_brick_edges(n):
    nx, ny, nz = n
    shape = (nz, ny, nx)
    rng = np.random.default_rng(nx + 100 * ny + 10000 * nz)
    theta = (nn.init_params(7) + 0.02 * rng.standard_normal(nn.num_params())).astype(np.float32)
    inp = nn.bf16_round(rng.standard_normal(shape + (4,)))
    target = rng.standard_normal(shape).astype(np.float32)
    x8 = np.zeros(shape + (8,), dtype=np.float32)
    x8[..., :4] = inp
    net = hp.Net(n, training=True)
    net.set_params(torch.from_numpy(theta).cuda())
    tgt = torch.from_numpy(target).cuda()
    x = torch.from_numpy(x8).cuda().to(torch.bfloat16).contiguous()
    losses, grads = [], []
    for _ in range(2):  # workspaces are reused by the next step
        losses.append(net.loss_grad_raw(x, tgt))
        grads.append(net.get_grad().cpu().numpy().astype(np.float64))
    net.close()
    assert losses[0] == losses[1] and np.array_equal(grads[0], grads[1])
    loss_r, g_r = nn.loss_and_grad(theta.astype(np.float64), inp, target.astype(np.float64), bf16=True)
    assert abs(losses[0] - loss_r) <= 5e-3 * loss_r
    at = 0
    for ci, co in nn.CONVS:
        for size in (27 * ci * co, co):
            a, b = grads[0][at:at + size], g_r[at:at + size]
            at += size
            norm = np.linalg.norm(b)
            assert np.linalg.norm(a - b) <= 3e-2 * norm, (ci, co, size)
            assert norm == 0 or a @ b >= 0.999 * np.linalg.norm(a) * norm, (ci, co, size)
    assert np.linalg.norm(grads[0][at:] - g_r[at:]) <= 3e-2 * np.linalg.norm(g_r[at:])

"""Training on grids whose weight gradients run on streams of their own, and on smaller ones.

The sums' order is fixed, so a step gives the same bits whenever and on whatever stream it runs: steps
with other work between them, on a stream of the caller's, and of two networks at once are compared with
the same steps run one at a time.
"""
import ctypes

import numpy as np
import pytest

from oracle import nn

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a HIP GPU")]

import paper_1112_3507_amd as hp  # noqa: E402


def inputs(n, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    x = torch.zeros(n[2], n[1], n[0], 8, device="cuda")
    x[..., :4] = torch.randn(n[2], n[1], n[0], 4, device="cuda", generator=gen)
    return x.to(torch.bfloat16).contiguous(), torch.randn(n[2], n[1], n[0], device="cuda", generator=gen)


def steps(net, data, count):
    out = []
    for k in range(count):
        net.loss_grad_raw(*data[k % len(data)])
        out.append(net.get_grad().clone())
        net.adam(1e-3)
    out.append(net.get_params().clone())
    return out


def same(a, b):
    torch.cuda.synchronize()
    return all(torch.equal(x, y) for x, y in zip(a, b))


@pytest.mark.parametrize("n", [(64, 64, 32), (64, 64, 28), (68, 36, 60)])
def test_steps_are_the_same_on_any_stream(n):
    theta = torch.from_numpy(nn.init_params(3).astype(np.float32)).cuda()
    data = [inputs(n, s) for s in (1, 2)]
    nets = [hp.Net(n, training=True) for _ in range(2)]
    for net in nets:
        net.set_params(theta)
    ref = steps(nets[0], data, 4)
    torch.cuda.synchronize()
    stream = torch.cuda.Stream()
    assert nets[1]._lib.hp_nn_set_stream(nets[1]._h, ctypes.c_void_p(stream.cuda_stream)) == 0
    other = torch.randn(2048, 2048, device="cuda")
    torch.cuda.synchronize()
    nets[0].set_params(theta)
    got = []
    with torch.cuda.stream(stream):
        for k in range(4):  # the second network's steps among the first one's and other work
            nets[1].loss_grad_raw(*data[k % 2])
            other = (other @ other).clamp(-1, 1)
            got.append(nets[1].get_grad().clone())
            nets[1].adam(1e-3)
            with torch.cuda.stream(torch.cuda.default_stream()):
                nets[0].loss_grad_raw(*data[k % 2])
        got.append(nets[1].get_params().clone())
    assert same(ref, got)
    for net in nets:
        net.close()

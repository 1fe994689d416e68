"""Weight gradients beside the rest of a training step: overlapping steps, and an order that can't be made.

Steps are enqueued several deep without the host reading anything (no loss is asked for), of two networks on streams of
their own at once, with other work among them; they have to give the bits of the same steps with the weight
gradients on the network's own stream. Where an event between the streams can't be recorded, the step has to end in
an error before anything unordered is launched, and the next one has to be right again.
"""
import ctypes

import numpy as np
import pytest

from oracle import nn

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a HIP GPU")]

import paper_1112_3507_amd as hp  # noqa: E402

ptr = lambda t: ctypes.c_void_p(t.data_ptr())  # noqa: E731


def inputs(n, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    x = torch.zeros(n[2], n[1], n[0], 8, device="cuda")
    x[..., :4] = torch.randn(n[2], n[1], n[0], 4, device="cuda", generator=gen)
    return x.to(torch.bfloat16).contiguous(), torch.randn(n[2], n[1], n[0], device="cuda", generator=gen)


def network(n, seed, beside):
    net = hp.Net(n, training=True)
    net.set_params(torch.from_numpy(nn.init_params(seed).astype(np.float32)).cuda())
    return net, switch(net, beside)


def switch(net, how):
    f = hp.load_library().hp_test_nn_beside
    f.argtypes, f.restype = [ctypes.c_void_p, ctypes.c_int], ctypes.c_int
    return f(net._h, how)


def step(net, data, grad):
    """One step with nothing read on the host; grad: where its gradient goes."""
    lib = net._lib
    assert lib.hp_nn_loss_grad_raw(net._h, ptr(data[0]), ptr(data[1]), None) == hp.OK
    assert lib.hp_nn_get_grad(net._h, ptr(grad)) == hp.OK
    assert lib.hp_nn_adam(net._h, 1e-3) == hp.OK


@pytest.mark.parametrize("n", [(64, 64, 32), (68, 36, 60), (64, 128, 64)])
def test_overlapping_steps_equal_steps_in_one_stream(n):
    count = 4
    data = [inputs(n, s) for s in (1, 2, 3)]
    grads = lambda: [torch.full((hp.num_params(),), float("nan"), device="cuda") for _ in range(count)]  # noqa: E731
    want = []
    for seed in (3, 4):
        net, has_streams = network(n, seed, 0)
        assert has_streams
        want.append(grads())
        for k in range(count):
            step(net, data[(k + seed) % 3], want[-1][k])
            torch.cuda.synchronize()
        net.close()
    nets = [network(n, seed, 1)[0] for seed in (3, 4)]
    got = [grads(), grads()]
    other = torch.randn(2048, 2048, device="cuda")
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    for net, stream in zip(nets, streams):
        assert net._lib.hp_nn_set_stream(net._h, ctypes.c_void_p(stream.cuda_stream)) == hp.OK
    for k in range(count):
        for q, seed in enumerate((3, 4)):
            step(nets[q], data[(k + seed) % 3], got[q][k])
        other = (other @ other).clamp(-1, 1)
    torch.cuda.synchronize()
    for q in range(2):
        for k in range(count):
            assert torch.equal(got[q][k], want[q][k]), (q, k)
        nets[q].close()


def test_a_step_whose_streams_cannot_be_ordered_ends_in_an_error():
    n = (64, 64, 32)
    data = inputs(n, 1)
    net, _ = network(n, 3, 1)
    want = torch.empty(hp.num_params(), device="cuda")
    got = torch.empty_like(want)
    net.loss_grad_raw(*data)
    assert net._lib.hp_nn_get_grad(net._h, ptr(want)) == hp.OK
    before = net.get_params()
    torch.cuda.synchronize()
    switch(net, 2)
    assert net._lib.hp_nn_loss_grad_raw(net._h, ptr(data[0]), ptr(data[1]), None) == hp.EHIP
    assert b"event" in net._lib.hp_nn_last_error()
    assert torch.equal(net.get_params(), before)
    switch(net, 1)
    net.loss_grad_raw(*data)
    assert net._lib.hp_nn_get_grad(net._h, ptr(got)) == hp.OK
    torch.cuda.synchronize()
    assert torch.equal(got, want)
    net.close()

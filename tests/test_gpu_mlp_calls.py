"""Calls of the warm-start network beside each other: threads, buffers, memory."""
import threading

import numpy as np
import pytest

from oracle import mlp as omlp
from paper_0711_0999_amd import inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")   # before the library initializes the device


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def test_networks_of_two_widths_of_input_in_two_threads(lib):
    """One kernel serves both networks, with different LDS sizes: no call may
    take away what the other's launch needs."""
    print("case: BF16 forward of two networks in two threads", flush=True)
    nets, xs, want = [], [], []
    for d_in in (33, 576):
        shapes = omlp.layer_shapes(d_in, 128, 2, 2)
        xs.append(dev(inputs.random_rows(70, d_in, seed=d_in + 1)))
        nets.append(lib.MLP(d_in, 128, 2, 2, params=inputs.network_params(shapes, seed=d_in)))
        want.append(nets[-1].forward(xs[-1], bf16=True).cpu().numpy())
    failed = []

    def work(q):
        try:
            for _ in range(2000):
                y = nets[q].forward(xs[q], bf16=True)
            if not np.array_equal(y.cpu().numpy(), want[q]):
                failed.append((q, "other values"))
        except Exception as e:      # a refused launch
            failed.append((q, e))

    threads = [threading.Thread(target=work, args=(q,)) for q in (0, 1)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for net in nets:
        net.close()
    assert not failed


@pytest.mark.parametrize("at", [0, 1, -1])
@pytest.mark.parametrize("d_in,d_out", [(96, 2), (16, 16)])
def test_bf16_outputs_that_overlap_the_inputs(lib, d_in, d_out, at):
    """y in x's own memory, at its start, its middle and its end: every input is
    read before any output is written."""
    print(f"case: BF16 forward into its inputs, {d_in} -> {d_out}, at {at}", flush=True)
    rows = 40000
    shapes = omlp.layer_shapes(d_in, 128, 3, d_out)
    x = dev(inputs.random_rows(rows, d_in, seed=21))
    net = lib.MLP(d_in, 128, 3, d_out, params=inputs.network_params(shapes, seed=22))
    want = net.forward(x, bf16=True).cpu().numpy()
    first = {0: 0, 1: rows * (d_in - d_out) // 2, -1: rows * (d_in - d_out)}[at]
    y = x.view(-1)[first:first + rows * d_out]
    net._check(net._lib.fk_mlp_forward(net._h, x.data_ptr(), rows, y.data_ptr(), 1), "forward")
    assert np.array_equal(y.cpu().numpy().reshape(rows, d_out), want)
    net.close()


def test_evaluation_allocates_no_gradient_parts(lib):
    """FP32 rows through 17 layers of 512 x 512: the activations and deltas of
    2048 rows are 21 buffers of 4 MiB; the gradient's parts would be 17 of 16."""
    print("case: memory of an FP32 evaluation", flush=True)
    shapes = omlp.layer_shapes(96, 512, 18, 2)
    x = dev(inputs.random_rows(2048, 96, seed=31))
    net = lib.MLP(96, 512, 18, 2, params=inputs.network_params(shapes, seed=32))
    y = net.forward(x[:1].contiguous())
    free = torch.cuda.mem_get_info()[0]
    y = net.forward(x)
    torch.cuda.synchronize()
    assert free - torch.cuda.mem_get_info()[0] < 160 * 2 ** 20
    # the parts come with the first gradient, and again with more rows
    t = dev(inputs.random_rows(2048, 2, seed=33))
    for rows in (100, 2048, 700):
        got = net.loss_grad(x[:rows].contiguous(), t[:rows].contiguous())
        other = lib.MLP(96, 512, 18, 2, params=net.get_params())
        want = other.loss_grad(x[:rows].contiguous(), t[:rows].contiguous())
        other.close()
        assert got[0] == want[0] and np.array_equal(got[1], want[1])
    assert np.array_equal(net.forward(x).cpu().numpy(), y.cpu().numpy())
    net.close()


def test_gradient_of_a_layer_beyond_two_to_the_31(lib):
    """65,537 x 32,768 weights in one layer; numbers for which every product and
    sum is exact."""
    print("case: gradient of a layer of 2^31 + 32768 weights", flush=True)
    d_in, width = 32768, 65537
    x = np.ones((1, d_in), np.float32)
    x[0, 1::2] = 2.0
    xd, td = dev(x), dev(np.full((1, 1), -0.5, np.float32))
    n1 = width * d_in
    p = np.zeros(n1 + 2 * width + 1, np.float32)   # W1 = b1 = 0: h = 0, y = b2 = 0
    w2 = (1.0 + np.arange(width) % 5).astype(np.float32)
    p[n1 + width:n1 + 2 * width] = w2
    net = lib.MLP(d_in, width, 2, 1, params=p)
    del p
    loss, g = net.loss_grad(xd, td)
    net.close()
    assert loss == 0.25                            # d = 2 (0 + 0.5) = 1
    assert np.array_equal(g[n1:n1 + width], w2)
    assert not g[n1 + width:n1 + 2 * width].any() and g[-1] == 1.0
    for o in (0, 1, 32768, width - 2, width - 1):
        assert np.array_equal(g[o * d_in:(o + 1) * d_in], w2[o] * x[0])


def test_bf16_forward_of_the_most_rows(lib):
    """2^31 - 1 rows of one input: more threads than one launch can have."""
    print("case: BF16 forward of 2^31 - 1 rows", flush=True)
    rows = 2 ** 31 - 1
    shapes = omlp.layer_shapes(1, 128, 2, 1)
    net = lib.MLP(1, 128, 2, 1, params=inputs.network_params(shapes, seed=41))
    x = torch.arange(rows, dtype=torch.int32, device="cuda").remainder_(1009).float()
    x = x.div_(500.0).view(rows, 1)
    y = net.forward(x, bf16=True).view(-1)
    want = net.forward(x[:1009].contiguous(), bf16=True).view(-1)
    for q in range(0, rows, 1009 * 2 ** 18):
        part = y[q:q + 1009 * 2 ** 18]
        assert torch.equal(part, want.repeat(-(-len(part) // 1009))[:len(part)])
    net.close()


@pytest.mark.parametrize("d_in,width,depth,d_out,rows", [
    (96, 512, 4, 2, 1000), (33, 128, 2, 16, 65), (64, 256, 3, 1, 63), (20, 384, 2, 5, 129)])
def test_fused_evaluation_equals_layer_by_layer(lib, d_in, width, depth, d_out, rows):
    """With zeros as inputs 577 wide the same network goes layer by layer: the same
    depths in the same order, bit for bit."""
    print(f"case: fused and layered BF16, {d_in} -> {width} x {depth - 1} -> {d_out}",
          flush=True)
    shapes = omlp.layer_shapes(d_in, width, depth, d_out)
    p = inputs.network_params(shapes, seed=51)
    x = inputs.random_rows(rows, d_in, seed=52)
    w1 = np.zeros((width, 577), np.float32)
    w1[:, :d_in] = p[:width * d_in].reshape(width, d_in)
    x2 = np.zeros((rows, 577), np.float32)
    x2[:, :d_in] = x
    xd, x2d = dev(x), dev(x2)
    net = lib.MLP(d_in, width, depth, d_out, params=p)
    wide = lib.MLP(577, width, depth, d_out,
                   params=np.concatenate([w1.ravel(), p[width * d_in:]]))
    y, y2 = net.forward(xd, bf16=True), wide.forward(x2d, bf16=True)
    assert np.array_equal(y.cpu().numpy(), y2.cpu().numpy())
    net.close()
    wide.close()

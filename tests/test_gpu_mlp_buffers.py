"""Caller's buffers of the network's passes that share memory: outputs over the
inputs, d loss / d X over d loss / d yhat.  Bit for bit as with buffers apart, in the
whole-pass kernels (several workgroups of 16 rows) and in the launches per product."""
import ctypes as C

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes", [(1, 33, 1), (3, 40, 17, 1), (15, 256, 256, 256, 1), (4, 1),
                                   (2, 2112, 1)])
def test_buffers_that_share_memory(sizes):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2507_06938_amd import dalia as D
    n, d = 1000, sizes[0]
    net = D.MLP(sizes, max_batch=n)
    g = torch.Generator(device="cuda").manual_seed(1)
    net.params.normal_(0, 0.3, generator=g)
    X = torch.randn(n, d, device="cuda", generator=g)
    dy = torch.randn(n, device="cuda", generator=g)
    y0 = net.forward(X).clone()
    dX0 = net.backward(dy, want_dx=True).clone()
    g0 = net.grads.clone()
    for shift in sorted({0, n * (d - 1) // 2, n * (d - 1)}):
        buf = X.clone()
        out = buf.view(-1)[shift:shift + n]
        net.forward(buf, out=out)
        assert torch.equal(out, y0), shift
        buf = torch.zeros(n * d, device="cuda")
        buf[shift:shift + n] = dy
        D._check("mlp_bwd", D.lib().mlp_bwd(net.h, C.c_void_p(buf.data_ptr() + 4 * shift), n,
                                            C.c_void_p(buf.data_ptr()), D._stream()))
        torch.cuda.synchronize()
        assert torch.equal(buf.view(n, d), dX0), shift
        assert np.array_equal(net.grads.cpu().numpy(), g0.cpu().numpy()), shift


def test_a_narrower_network_leaves_a_wide_one_its_lds():
    """The kernels' limit of dynamic LDS belongs to the function: networks of
    several widths beyond 64 KB of it, created in any order."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2507_06938_amd import dalia as D
    X = torch.randn(20, 3, device="cuda")
    dy = torch.randn(20, device="cuda")
    nets = [D.MLP((3, h, 1), max_batch=64) for h in (2048, 1100, 1030)]
    for net in nets:
        net.params.normal_(0, 0.1)
    want = [(net.forward(X).clone(), net.backward(dy, want_dx=True).clone()) for net in nets[::-1]]
    nets.append(D.MLP((3, 1040, 1), max_batch=64))
    got = [(net.forward(X).clone(), net.backward(dy, want_dx=True).clone()) for net in nets[2::-1]]
    for a, b in zip(want, got):
        assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])
        assert torch.isfinite(a[0]).all() and a[0].abs().max() > 0

"""The whole-pass network kernels at the edges of their tiles (rows in groups
of 16, columns in blocks of 16, k in 32s and 256s) and the launch-per-product
path of wider networks, against the FP64 reference with the same bfloat16
rounding points."""
import math

import numpy as np
import pytest

from oracle import mlp as OL

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _rel(a, b):
    return np.linalg.norm(np.asarray(a) - np.asarray(b)) / max(np.linalg.norm(b), 1e-30)


@pytest.mark.parametrize("sizes", [(1, 1), (3, 16, 1), (15, 17, 31, 1), (7, 40, 300, 33, 1),
                                   (15, 256, 256, 256, 1), (4, 272, 520, 1), (20, 1000, 1),
                                   (5, 2112, 1)])
@pytest.mark.parametrize("n", [1, 16, 17, 130])
def test_passes(sizes, n):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2507_06938_amd import dalia as D
    rng = np.random.default_rng(sum(sizes) + n)
    params = [(rng.standard_normal((o, i)).astype(np.float32) / np.float32(math.sqrt(i)),
               (0.1 * rng.standard_normal(o)).astype(np.float32))
              for i, o in zip(sizes[:-1], sizes[1:])]
    net = D.MLP(sizes, max_batch=144)
    net.params.copy_(torch.from_numpy(np.concatenate(
        [np.concatenate([W.ravel(), b]) for W, b in params])))
    params = [(W.astype(np.float64), b.astype(np.float64)) for W, b in params]
    X = rng.standard_normal((n, sizes[0])).astype(np.float32)
    dy = rng.standard_normal(n).astype(np.float32)
    Xd = torch.from_numpy(X).cuda()
    yhat = net.forward(Xd)
    Xd.zero_()  # the backward pass reads the network's own copy
    dX = net.backward(torch.from_numpy(dy).cuda(), want_dx=True)
    torch.cuda.synchronize()
    grads = net.grads.cpu().numpy()
    ref_y, cache = OL.forward(params, X.astype(np.float64), bf16=True)
    ref_g, ref_dX = OL.backward(params, cache, dy.astype(np.float64), bf16=True)
    # rounding points alike, FP32 sums in another order: a value near a
    # bfloat16 tie may round the other way (2^-8 of it)
    scale = np.linalg.norm(ref_y) + math.sqrt(n)
    assert np.linalg.norm(yhat.cpu().numpy() - ref_y) <= 4e-3 * scale
    assert _rel(dX.cpu().numpy(), ref_dX) <= 1e-2
    off = 0
    for gW, gb in ref_g:
        assert _rel(grads[off:off + gW.size], gW.ravel()) <= 2e-2
        off += gW.size
        assert _rel(grads[off:off + gb.size], gb) <= 2e-2
        off += gb.size
    # without the input gradient the parameter gradients are the same
    net.forward(torch.from_numpy(X).cuda())
    net.backward(torch.from_numpy(dy).cuda())
    torch.cuda.synchronize()
    assert np.array_equal(net.grads.cpu().numpy(), grads)


# both sides of the lines between one launch a pass and one per product: rows 16 | 17
# at 600 columns, 32 | 33 at 1000 and (backward) at 1200 and with d loss / d X at 2048,
# 128 | 129 at 1800, 4096, 8192 and 16384 rows, a widest layer that is not the first
@pytest.mark.parametrize("sizes,n", [((3, 600, 1), 16), ((3, 600, 1), 17), ((3, 40, 1000, 1), 32),
                                     ((3, 40, 1000, 1), 33), ((3, 2048, 24, 1), 32),
                                     ((3, 2048, 24, 1), 33), ((3, 1200, 40, 1), 32),
                                     ((3, 1200, 40, 1), 33), ((3, 1800, 1), 128),
                                     ((3, 1800, 1), 129), ((3, 96, 1), 8192), ((3, 96, 1), 8193),
                                     ((3, 50, 1), 16385), ((2, 300, 1), 4097)])
def test_paths(sizes, n):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2507_06938_amd import dalia as D
    rng = np.random.default_rng(sum(sizes) + n)
    params = [(rng.standard_normal((o, i)).astype(np.float32) / np.float32(math.sqrt(i)),
               (0.1 * rng.standard_normal(o)).astype(np.float32))
              for i, o in zip(sizes[:-1], sizes[1:])]
    net = D.MLP(sizes, max_batch=n)
    net.params.copy_(torch.from_numpy(np.concatenate(
        [np.concatenate([W.ravel(), b]) for W, b in params])))
    params = [(W.astype(np.float64), b.astype(np.float64)) for W, b in params]
    X = rng.standard_normal((n, sizes[0])).astype(np.float32)
    dy = rng.standard_normal(n).astype(np.float32)
    yhat = net.forward(torch.from_numpy(X).cuda())
    net.backward(torch.from_numpy(dy).cuda())
    plain = net.grads.cpu().numpy().copy()
    dX = net.backward(torch.from_numpy(dy).cuda(), want_dx=True)
    torch.cuda.synchronize()
    ref_y, cache = OL.forward(params, X.astype(np.float64), bf16=True)
    ref_g, ref_dX = OL.backward(params, cache, dy.astype(np.float64), bf16=True)
    # the bounds of test_passes
    assert np.linalg.norm(yhat.cpu().numpy() - ref_y) <= 4e-3 * (np.linalg.norm(ref_y)
                                                                + math.sqrt(n))
    assert _rel(dX.cpu().numpy(), ref_dX) <= 1e-2
    for grads in (plain, net.grads.cpu().numpy()):
        off = 0
        for gW, gb in ref_g:
            assert _rel(grads[off:off + gW.size], gW.ravel()) <= 2e-2
            off += gW.size
            assert _rel(grads[off:off + gb.size], gb) <= 2e-2
            off += gb.size

"""The two wave arrangements of the 64 x 64 tile product (eight waves up to 4095
tiles a launch, four from 4096 on) on both sides of the line: the same bits for
the columns both compute, against a product by torch in FP64 (K eps of the
largest sum of magnitudes), with an odd K and a k range that is not a multiple
of a staged chunk."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def D():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2507_06938_amd import dalia
    dalia.lib()
    return dalia


@pytest.mark.parametrize("K", [16, 41, 88])
@pytest.mark.parametrize("tb", [0, 1])
def test_both_arrangements(D, K, tb):
    M, N = 4096, 4096  # 64 x 64 tiles of 64
    g = torch.Generator(device="cuda").manual_seed(K)
    A = torch.randn(K, M, generator=g, dtype=torch.float64, device="cuda")  # column-major M x K
    B = torch.randn(*((K, N) if tb else (N, K)), generator=g, dtype=torch.float64, device="cuda")
    out = []
    for n in (N, N - 64):
        C = torch.zeros(n, M, dtype=torch.float64, device="cuda")  # column-major M x n
        assert D.lib().dl_dgemm(0, tb, 0, M, n, K, 1.0, D._ptr(A), M, D._ptr(B), N if tb else K,
                                0.0, D._ptr(C), M, D._stream()) == 0
        out.append(C)
    torch.cuda.synchronize()
    Bt = B if tb else B.T  # K x N
    want = Bt.T.contiguous() @ A
    bound = K * 2.3e-16 * (Bt.abs().T.contiguous() @ A.abs()).max()
    assert (out[0] - want).abs().max() <= bound
    assert torch.equal(out[0][:N - 64], out[1])


@pytest.mark.parametrize("K", [41, 96])
def test_arrangements_of_a_nearly_full_round(D, K):
    """One product of 768, 800, 1024 and 1088 equal tiles (eight, four, four, eight
    waves a tile): the same bits for the columns they share."""
    M = 2048
    g = torch.Generator(device="cuda").manual_seed(K)
    A = torch.randn(K, M, generator=g, dtype=torch.float64, device="cuda")
    B = torch.randn(2176, K, generator=g, dtype=torch.float64, device="cuda")
    out = []
    for n in (1536, 1600, 2048, 2176):
        C = torch.zeros(n, M, dtype=torch.float64, device="cuda")
        assert D.lib().dl_dgemm(0, 0, 0, M, n, K, 1.0, D._ptr(A), M, D._ptr(B), K, 0.0, D._ptr(C),
                                M, D._stream()) == 0
        out.append(C)
    torch.cuda.synchronize()
    bound = K * 2.3e-16 * (B.abs() @ A.abs()).max()
    assert (out[3] - B @ A).abs().max() <= bound
    for C in out[:3]:
        assert torch.equal(C, out[3][:C.shape[0]])

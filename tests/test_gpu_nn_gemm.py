"""The bfloat16 product at the edges of its tiles (32 rows and columns, 64 of the depth), with every
transposition, with bases and leading dimensions that allow four values a load and that do
not, and with a depth split.  Operands are small whole numbers: every product and partial sum is exact in
float32, so results are compared exactly."""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def T():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2212_01253_amd import nn
    nn.lib()
    return nn


def operand(rows, cols, pad, off):
    """Array [rows][cols] of row length cols + pad in a buffer that is NaN elsewhere, `off` elements in."""
    v = torch.randint(-8, 9, (rows, cols), device="cuda").float()
    buf = torch.full((off + rows * (cols + pad),), float("nan"), dtype=torch.bfloat16, device="cuda")
    buf[off:].view(rows, cols + pad)[:, :cols] = v.bfloat16()
    return v.double(), buf.view(torch.int16)[off:]


@pytest.mark.parametrize("ta", [0, 1])
@pytest.mark.parametrize("tb", [0, 1])
@pytest.mark.parametrize("M,N,K,pad,off", [
    (1, 1, 1, 0, 0), (31, 33, 63, 1, 1), (32, 32, 64, 0, 0), (33, 31, 65, 0, 4), (64, 96, 128, 4, 0),
    (65, 1, 192, 4, 1), (1, 70, 200, 3, 0), (100, 40, 7, 1, 4), (256, 64, 768, 0, 0)])
def test_gemm_exact(T, M, N, K, pad, off, ta, tb):
    A, a16 = operand(*((K, M) if ta else (M, K)), pad, off)
    B, b16 = operand(*((N, K) if tb else (K, N)), pad, off)
    ref = ((A.t() if ta else A) @ (B.t() if tb else B)).float()
    lda, ldb, ldc = (M if ta else K) + pad, (K if tb else N) + pad, N + 3
    C = torch.full((M, ldc), 2.0, device="cuda")
    T.gemm(M, N, K, a16, lda, ta, b16, ldb, tb, C, ldc, beta=1.0)
    assert torch.equal(C[:, :N], ref + 2) and (C[:, N:] == 2).all()
    parts = torch.empty(3 * M * N, device="cuda")
    C.fill_(2.0)
    T.gemm_splitk(M, N, K, a16, lda, ta, b16, ldb, tb, C, ldc, 3, parts)
    assert torch.equal(C[:, :N], ref) and (C[:, N:] == 2).all()

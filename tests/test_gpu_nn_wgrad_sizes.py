"""Weight gradients of the longest rows and of the most channels: sums of zeros and ones, whole numbers
below 2^24, which every order of summation gives exactly."""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nn():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2212_01253_amd import nn
    yield nn
    torch.cuda.empty_cache()


@pytest.mark.parametrize("s,W,xbf16", [(1, 1 << 29, True), (1, (1 << 29) + 2, True), (1, 400_000_000, False), (2, 1 << 29, True)])
def test_long_rows(nn, s, W, xbf16):
    x = torch.zeros((s, W), dtype=torch.bfloat16 if xbf16 else torch.float32, device="cuda")
    dy = torch.zeros(W // s, dtype=torch.bfloat16, device="cuda")
    x[0, ::97] = 1
    x[-1, ::83] = 1
    x[:, -1] = 1
    dy[::89] = 1
    dy[-1] = 1
    dw = torch.full((1, 1, 3, 3), -1.0, device="cuda")
    nn.conv3x3_weight_grad(1, 1, 1, s, W, s, dy.view(torch.int16), x.view(torch.int16) if xbf16 else x, dw, 64,
                           torch.zeros(64 * 9, device="cuda"))
    at = dy.nonzero()[:, 0]
    for i in range(3):       # the one gradient row meets input rows -1, 0, 1
        for j in range(3):
            p = s * at + j - 1
            p = p[(p >= 0) & (p < W)]
            ref = float((x[i - 1][p] != 0).sum()) if 0 <= i - 1 < s else 0.0
            assert float(dw[0, 0, i, j]) == ref


@pytest.mark.parametrize("Co,C", [(8192, 16384), (8191, 3800)])
def test_many_channels(nn, Co, C):
    # one pixel: the middle tap is the product of the two channels, the others have none
    x = (torch.arange(C, device="cuda") % 3 == 1).to(torch.bfloat16)
    dy = (torch.arange(Co, device="cuda") % 5 < 2).to(torch.bfloat16)
    dw = torch.full((Co, C, 3, 3), -1.0, device="cuda")
    nn.conv3x3_weight_grad(Co, C, 1, 1, 1, 1, dy.view(torch.int16), x.view(torch.int16), dw, 1,
                           torch.empty(Co * C * 9, device="cuda"))
    torch.cuda.synchronize()
    assert torch.equal(dw[:, :, 1, 1], dy.float()[:, None] * x.float()[None])
    dw[:, :, 1, 1] = 0
    assert not bool(dw.any())

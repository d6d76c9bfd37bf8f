"""Convolutions around the sizes where the dispatch leaves the register rows for halo tiles: the most product
rows a launch has blocks for, and 2^26 pixels.  Both kernels add the taps of a channel chunk in the same
order, so pixels and channels of the two are compared bit for bit (tolerance 0)."""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

MOST = 65535 * 64


@pytest.fixture(scope="module")
def nn():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2212_01253_amd import nn
    yield nn
    torch.cuda.empty_cache()


def randn16(gen, *s):
    return torch.randn(s, device="cuda", generator=gen).to(torch.bfloat16)


@pytest.mark.parametrize("M", [MOST, MOST + 40])
def test_many_output_channels(nn, M):
    gen = torch.Generator(device="cuda").manual_seed(1)
    x, w = randn16(gen, 1, 1, 2, 18), randn16(gen, M, 9)
    y = torch.zeros((M, 1, 2, 18), device="cuda")
    nn.conv3x3(M, 1, 1, 2, 18, 1, w.view(torch.int16), x.view(torch.int16), y)
    for a, b in ((0, 100), (M - 100, M)):
        part = torch.zeros((100, 1, 2, 18), device="cuda")
        nn.conv3x3(100, 1, 1, 2, 18, 1, w[a:b].contiguous().view(torch.int16), x.view(torch.int16), part)
        assert torch.equal(y[a:b], part)


@pytest.mark.parametrize("C,s", [(MOST, 1), (MOST + 40, 1), (MOST // 4 + 10, 2)])
def test_many_input_channels(nn, C, s):
    gen = torch.Generator(device="cuda").manual_seed(2)
    dy, w = randn16(gen, 1, 1, 2, 18), randn16(gen, 1, C, 9)
    dx = torch.zeros((C, 1, 2 * s, 18 * s), device="cuda")
    nn.conv3x3_adjoint(1, C, 1, 2 * s, 18 * s, s, w.view(torch.int16), dy.view(torch.int16), dx)
    for a, b in ((0, 100), (C - 100, C)):
        part = torch.zeros((100, 1, 2 * s, 18 * s), device="cuda")
        nn.conv3x3_adjoint(1, 100, 1, 2 * s, 18 * s, s, w[:, a:b].contiguous().view(torch.int16), dy.view(torch.int16), part)
        assert torch.equal(dx[a:b], part)


@pytest.mark.parametrize("s", [1, 2])
@pytest.mark.parametrize("B", [1023, 1024])
def test_many_pixels(nn, B, s):
    gen = torch.Generator(device="cuda").manual_seed(3)
    x, w = randn16(gen, 2, B, 256, 256), randn16(gen, 3, 18)
    y = torch.zeros((3, B, 256 // s, 256 // s), dtype=torch.int16, device="cuda")
    nn.conv3x3(3, 2, B, 256, 256, s, w.view(torch.int16), x.view(torch.int16), y)
    dx = torch.zeros((2, B, 256, 256), device="cuda")
    nn.conv3x3_adjoint(3, 2, B, 256, 256, s, w.view(torch.int16), y, dx)
    for a in (0, B - 3):
        yp = torch.zeros((3, 3, 256 // s, 256 // s), dtype=torch.int16, device="cuda")
        nn.conv3x3(3, 2, 3, 256, 256, s, w.view(torch.int16), x[:, a:a + 3].contiguous().view(torch.int16), yp)
        assert torch.equal(y[:, a:a + 3], yp)
        dp = torch.zeros((2, 3, 256, 256), device="cuda")
        nn.conv3x3_adjoint(3, 2, 3, 256, 256, s, w.view(torch.int16), yp, dp)
        assert torch.equal(dx[:, a:a + 3], dp)

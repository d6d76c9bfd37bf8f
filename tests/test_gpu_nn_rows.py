"""3x3 convolutions (forward, input and weight gradient) at the edges of their tiles.

The reference is the sum over the nine taps in float64 of the same bfloat16 operands.  Each
output is a float32 sum of 9 C products (exact in float32) and a bias, so it is within
(9 C + 2) 2^-24 times the sum of the products' magnitudes, and a bfloat16 output within 2^-8 of its
magnitude (the unit roundoff) more.  Shapes cover rows shorter than a 32-pixel block and one over it,
columns that end inside a group of eight, one row, channel counts around the chunk of 16 and the
blocks of 32 and 64 and every tile shape of the dispatch (the large ones take 512 workgroups).  A weight
gradient is a float32 sum over the pixels, within their count (and the parts') times 2^-24 of the sum
of the magnitudes.
"""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def T():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2212_01253_amd import nn
    return nn


def conv64(x, w, s=1):
    """x [C][B][H][W], w [O][C][3][3] float64 -> [O][B][H / s][W / s], padding 1."""
    C, B, H, W = x.shape
    xp = torch.nn.functional.pad(x, (1, 1, 1, 1))
    y = torch.zeros((w.shape[0], B * (H // s) * (W // s)), dtype=torch.float64, device=x.device)
    for i in range(3):
        for j in range(3):
            y += w[:, :, i, j].contiguous() @ xp[:, :, i:i + H:s, j:j + W:s].reshape(C, -1)
    return y.reshape(-1, B, H // s, W // s)


def adjoint64(dy, w, s):
    """Input gradient of conv64: the stride-1 adjoint of dy spread onto every s-th pixel."""
    O, B, H, W = dy.shape
    d = torch.zeros((O, B, s * H, s * W), dtype=torch.float64, device=dy.device)
    d[:, :, ::s, ::s] = dy
    return conv64(d, w.flip(2, 3).transpose(0, 1).contiguous())


def shifted(t, by):
    """A copy of t whose storage starts `by` elements into an aligned buffer."""
    buf = torch.zeros(t.numel() + by, dtype=t.dtype, device=t.device)
    v = buf[by:].view(t.shape)
    v.copy_(t)
    return v


@pytest.mark.parametrize("O,C,B,H,W,s", [
    (1, 2, 1, 2, 34, 2), (33, 17, 1, 6, 66, 2), (64, 15, 2, 10, 64, 2), (31, 33, 1, 8, 130, 2), (70, 16, 2, 12, 48, 2),
    (40, 3, 32, 126, 128, 2), (3, 40, 33, 124, 96, 2),
    (1, 1, 1, 1, 17, 1), (32, 16, 2, 9, 18, 1), (33, 17, 1, 8, 31, 1), (31, 15, 2, 10, 32, 1), (64, 33, 1, 5, 33, 1), (65, 2, 3, 7, 34, 1),
    (5, 48, 1, 12, 48, 1), (70, 20, 1, 6, 95, 1), (96, 64, 1, 4, 130, 1), (16, 130, 1, 3, 64, 1), (128, 31, 1, 17, 24, 1),
    (40, 3, 32, 64, 64, 1), (34, 5, 64, 61, 20, 1), (9, 65, 32, 61, 98, 1)])
@pytest.mark.parametrize("xbf16,ybf16,shift", [(True, True, 0), (False, True, 0), (True, False, 1), (False, True, 1)])
def test_rows_convolution(T, O, C, B, H, W, s, xbf16, ybf16, shift):
    gen = torch.Generator(device="cuda").manual_seed(O * 1000 + C)
    rn = lambda *s: torch.randn(s, device="cuda", generator=gen)  # noqa: E731
    x, w, bias = rn(C, B, H, W), (rn(O, C, 3, 3) / (3 * C ** 0.5)).to(torch.bfloat16), rn(O)
    xb = x.to(torch.bfloat16)
    arg = shifted(xb.view(torch.int16) if xbf16 else x, shift)
    y = shifted(torch.zeros((O, B, H // s, W // s), dtype=torch.int16 if ybf16 else torch.float32, device="cuda"), shift)
    w16 = w.view(torch.int16).reshape(-1)
    T.conv3x3(O, C, B, H, W, s, w16, arg, y, bias=bias, relu=True)
    ref = conv64(xb.double(), w.double(), s) + bias.double().view(-1, 1, 1, 1)
    mag = conv64(xb.double().abs(), w.double().abs(), s) + bias.double().abs().view(-1, 1, 1, 1)
    tol = (9 * C + 2) * 2.0 ** -24 * mag + (2.0 ** -8 * ref.abs() if ybf16 else 0.0)
    got = (y.contiguous().view(torch.bfloat16) if ybf16 else y).double()
    assert bool(((got - torch.relu(ref)).abs() <= tol).all())
    # the input gradient, alone and added onto another
    dy = rn(O, B, H // s, W // s).to(torch.bfloat16)
    dy16 = shifted(dy.view(torch.int16), shift)
    ref, mag = adjoint64(dy.double(), w.double(), s), adjoint64(dy.double().abs(), w.double().abs(), s)
    base = rn(C, B, H, W)
    dx = shifted(base, shift)
    T.conv3x3_adjoint(O, C, B, H, W, s, w16, dy16, dx)
    tol = (9 * O + 2) * 2.0 ** -24 * mag
    assert bool(((dx.double() - ref).abs() <= tol).all())
    if shift % 2 == 0:   # (accumulation asks for 8-byte alignment)
        acc = base.clone()
        T.conv3x3_adjoint(O, C, B, H, W, s, w16, dy16, acc, accumulate=True)
        assert torch.equal(acc, base + dx)


@pytest.mark.parametrize("s", [1, 2])
@pytest.mark.parametrize("O,C,B,H,W,splits", [
    (1, 1, 1, 1, 1, 1), (2, 3, 1, 3, 2, 4), (33, 31, 2, 5, 33, 3), (32, 32, 1, 4, 16, 1), (31, 65, 3, 37, 31, 64),
    (64, 16, 1, 33, 64, 7), (5, 40, 2, 66, 40, 2), (70, 2, 1, 9, 95, 2048), (3, 7, 2, 130, 8, 16)])   # the gradient's H, W
@pytest.mark.parametrize("xbf16,shift", [(True, 0), (False, 0), (True, 1), (False, 1)])
def test_rows_weight_gradient(T, O, C, B, H, W, splits, s, xbf16, shift):
    gen = torch.Generator(device="cuda").manual_seed(O * 1000 + C)
    x = torch.randn((C, B, s * H, s * W), device="cuda", generator=gen)
    dy = torch.randn((O, B, H, W), device="cuda", generator=gen).to(torch.bfloat16)
    xb = x.to(torch.bfloat16)
    arg = shifted(xb.view(torch.int16) if xbf16 else x, shift)
    dw = torch.full((O, C, 3, 3), float("nan"), device="cuda")
    parts = torch.full((splits * O * C * 9,), float("nan"), device="cuda")
    T.conv3x3_weight_grad(O, C, B, s * H, s * W, s, shifted(dy.view(torch.int16), shift), arg, dw, splits, parts)

    def ref(a, b):
        ap, n = torch.nn.functional.pad(a, (1, 1, 1, 1)), B * H * W
        taps = [ap[:, :, i:i + s * H:s, j:j + s * W:s].reshape(C, n).t().contiguous() for i in range(3) for j in range(3)]
        return torch.stack([b.reshape(O, n) @ t for t in taps], dim=2).reshape(O, C, 3, 3)

    r, mag = ref(xb.double(), dy.double()), ref(xb.double().abs(), dy.double().abs())
    assert bool(((dw.double() - r).abs() <= (B * H * W + splits) * 2.0 ** -24 * mag).all())

"""Infinities and NaN of the input in a convolution's weight gradient: by definition the first and last
row and column of an image do not meet every tap, and the taps they do not meet stay as they are.

The reference is the sum of each tap's products in float64 over the same bfloat16 operands, where a value that
is not finite reaches only the sums it is part of; finite sums within their count times 2^-24 of the
sum of the magnitudes.  Heights and widths cover one unit and several, and strips that end in the middle of
a group of eight, at its end and at their own end."""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("s", [1, 2])
@pytest.mark.parametrize("H,W", [(4, 16), (5, 33), (9, 40), (37, 24), (70, 64), (66, 31), (3, 7), (40, 48)])   # the gradient's
@pytest.mark.parametrize("xbf16", [True, False])
@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
def test_taps_that_do_not_meet_stay_finite(H, W, s, xbf16, bad):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2212_01253_amd import nn
    O, C, B, splits = 33, 6, 2, 8
    gen = torch.Generator(device="cuda").manual_seed(H * 100 + W)
    x = torch.randn((C, B, s * H, s * W), device="cuda", generator=gen)
    x[0, 1, -1, W // 2] = bad    # last row, first row, last column, first column, a corner; channel 5 stays finite
    x[1, 0, 0, W // 2] = bad
    x[2, 1, H // 2, -1] = bad
    x[3, 0, H // 2, 0] = bad
    x[4, 1, -1, -1] = bad
    dy = torch.randn((O, B, H, W), device="cuda", generator=gen).to(torch.bfloat16)
    xb = x.to(torch.bfloat16)
    dw = torch.zeros((O, C, 3, 3), device="cuda")
    nn.conv3x3_weight_grad(O, C, B, s * H, s * W, s, dy.view(torch.int16), xb.view(torch.int16) if xbf16 else x, dw, splits,
                           torch.zeros(splits * O * C * 9, device="cuda"))
    n = B * H * W
    ap = torch.nn.functional.pad(xb.double(), (1, 1, 1, 1))
    for i in range(3):
        for j in range(3):
            t = ap[:, :, i:i + s * H:s, j:j + s * W:s].reshape(C, n)
            for c in range(C):
                got = dw[:, c, i, j].double()
                if not bool(torch.isfinite(t[c]).all()):
                    assert not bool(torch.isfinite(got).any()), (i, j, c)
                    continue
                r = (dy.double().reshape(O, n) * t[c]).sum(1)
                mag = (dy.double().reshape(O, n) * t[c]).abs().sum(1)
                assert bool(((got - r).abs() <= (n + splits) * 2.0 ** -24 * mag).all()), (i, j, c)

"""Input gradients added onto another: stride 1 into arrays of any alignment, stride 2 into 8-byte aligned ones
(others are refused).  The sum is one float32 addition per value, so it is compared bit for bit."""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("O,C,B,H,W,s", [(33, 17, 1, 8, 31, 1), (64, 33, 1, 5, 33, 1), (5, 48, 1, 12, 48, 1), (40, 3, 32, 64, 64, 1),
                                         (7, 5, 2, 9, 12, 1), (33, 17, 1, 6, 66, 2), (64, 15, 2, 10, 64, 2), (7, 5, 2, 10, 24, 2)])
@pytest.mark.parametrize("shift", [0, 1, 2, 3])
def test_accumulate(O, C, B, H, W, s, shift):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2212_01253_amd import msl, nn
    gen = torch.Generator(device="cuda").manual_seed(O * 1000 + C)
    rn = lambda *s: torch.randn(s, device="cuda", generator=gen)  # noqa: E731
    w16 = rn(O, C * 9).to(torch.bfloat16).view(torch.int16).reshape(-1)
    dy16 = rn(O, B, H // s, W // s).to(torch.bfloat16).view(torch.int16)
    base = rn(C, B, H, W)
    plain = torch.zeros_like(base)
    nn.conv3x3_adjoint(O, C, B, H, W, s, w16, dy16, plain)
    buf = torch.zeros(base.numel() + 4, device="cuda")
    dx = buf[shift:shift + base.numel()].view(base.shape)
    dx.copy_(base)
    if s == 2 and shift % 2:
        with pytest.raises(msl.MslError):
            nn.conv3x3_adjoint(O, C, B, H, W, s, w16, dy16, dx, accumulate=True)
        return
    nn.conv3x3_adjoint(O, C, B, H, W, s, w16, dy16, dx, accumulate=True)
    assert torch.equal(dx, base + plain)

"""2x upsampling and its adjoint over row widths and base offsets around the grouped
accesses (rows of whole 8-byte groups in aligned arrays) against the same copies and
sums in PyTorch: copies are equal, and the adjoint's four terms are added in one order,
so both are compared exactly."""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def T():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2212_01253_amd import nn
    return nn


@pytest.mark.parametrize("W", [1, 2, 3, 4, 6, 8, 10, 129, 256])
@pytest.mark.parametrize("xo,yo", [(0, 0), (1, 0), (0, 1), (2, 2), (4, 8)])
def test_upsample_exact(T, W, xo, yo):
    C, B, H = 3, 2, 5
    n = C * B * H * W
    for dt in (torch.bfloat16, torch.float32):
        x = torch.randn(n + xo, device="cuda").to(dt)
        y = torch.full((4 * n + yo + 8,), 7.0, device="cuda", dtype=dt)
        raw = (lambda t: t.view(torch.int16)) if dt == torch.bfloat16 else (lambda t: t)
        T.upsample2(C, B, H, W, raw(x)[xo:], raw(y)[yo:])
        ref = x[xo:].view(C * B * H, W).repeat_interleave(2, 0).repeat_interleave(2, 1)
        assert torch.equal(y[yo:yo + 4 * n].view(2 * C * B * H, 2 * W), ref)
        assert (y[:yo] == 7).all() and (y[yo + 4 * n:] == 7).all()
    dy = torch.randn(4 * n + xo, device="cuda")
    dx = torch.full((n + yo + 8,), 7.0, device="cuda")
    T.upsample2_adjoint(C, B, H, W, dy[xo:], dx[yo:])
    q = dy[xo:].view(C * B * H, 2, W, 2)
    ref = (q[:, 0, :, 0] + q[:, 0, :, 1]) + (q[:, 1, :, 0] + q[:, 1, :, 1])
    assert torch.equal(dx[yo:yo + n].view(-1, W), ref)
    assert (dx[:yo] == 7).all() and (dx[yo + n:] == 7).all()

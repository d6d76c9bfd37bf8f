"""The dataflow schedule of the exact propagator (two passes per slice) and of the forward
without a slice pack, against one launch per pass: the same arithmetic in the same order,
so every output is compared bit for bit (tolerance 0).

Slice counts go from below the fewest passes a launch takes, checkpoint intervals put
segment ends at odd and even slices, and the grids cover lines of one and of two wavefronts,
shorter than a wavefront, and axes of different line counts."""
import math

import pytest

from paper_2212_01253_amd import synth

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.fixture()
def M():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2212_01253_amd import msl
    msl.lib()
    yield msl
    msl.set_schedule(0)


def case(ny, nz, ns, exact):
    g = synth.Geometry(ny, nz, ns, 1.0, 0.9, 5.0, 0.1, math.radians(0.25), exact)
    gen = torch.Generator(device="cuda").manual_seed(7)
    d = 3e-5 * torch.rand((ns, ny, nz), device="cuda", generator=gen)
    ph = 0.1 * torch.rand((ny, nz), device="cuda", generator=gen)
    return g, d, d / 20, torch.polar(1.0 + 0.1 * torch.rand((ny, nz), device="cuda", generator=gen), ph)


GRIDS = [(16, 16, 9, 4), (16, 512, 12, 7), (512, 16, 11, 3), (32, 64, 33, 32), (64, 64, 2, 1), (64, 64, 1, 1),
         (64, 32, 40, 9), (128, 256, 37, 8), (256, 128, 70, 64), (256, 512, 19, 6), (512, 256, 18, 7),
         (512, 512, 12, 5), (512, 512, 7, 1)]


@pytest.mark.parametrize("ny,nz,ns,k", GRIDS)
def test_exact_bitwise_equal_to_per_pass(M, ny, nz, ns, k):
    g, d, b, probe = case(ny, nz, ns, 1)
    def gradient(ws):
        f, ck = M.forward(g, d, b, probe, ckpt_every=k, ws=ws)
        M.workspace_status(ws)
        gd, gb, gp = M.adjoint(g, d, b, ck, k, 0.5 * f, ws=ws)
        M.workspace_status(ws)
        return [f, ck, gd, gb, gp]

    M.set_schedule(1)
    ref = [x.clone() for x in gradient(M.workspace(g, k))]
    M.set_schedule(0)
    ws = M.workspace(g, k)
    ws.view(torch.uint8).fill_(0xFF)
    for _ in range(2):
        for r, o in zip(ref, gradient(ws)):
            assert torch.equal(r, o)


@pytest.mark.parametrize("exact", [0, 1])
@pytest.mark.parametrize("ny,nz,ns,k", GRIDS)
def test_noalloc_bitwise_equal_to_per_pass(M, ny, nz, ns, k, exact):
    g, d, b, probe = case(ny, nz, ns, exact)
    M.set_schedule(1)
    ref = [x.clone() for x in M.forward_noalloc(g, d, b, probe, k)]
    own = [x.clone() for x in M.forward_noalloc(g, d, b)[:1]]
    M.set_schedule(0)
    for _ in range(2):
        for r, o in zip(ref, M.forward_noalloc(g, d, b, probe, k)):
            assert torch.equal(r, o)
        assert torch.equal(own[0], M.forward_noalloc(g, d, b)[0])

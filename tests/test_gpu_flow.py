"""The one-launch (dataflow) schedule of the middle passes against one launch per pass.

Both run the same arithmetic in the same order, so every output is compared
bit for bit (tolerance 0).  Grids cover one-wavefront and two-wavefront workgroups,
square and not, lines shorter than a wavefront, line counts that differ between
the two pass axes (workgroups that sit passes out) and the smallest and largest
grid; slice counts and checkpoint intervals put the first and last pass of a launch on
either axis and go below the fewest passes a launch takes.
"""
import math
import threading

import numpy as np
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


def case(ny, nz, ns, seed=5):
    g = synth.Geometry(ny, nz, ns, 1.0, 1.0, 5.0, 0.1, math.radians(0.25), 0)
    gen = torch.Generator(device="cuda").manual_seed(seed)
    d = 3e-5 * torch.rand((ns, ny, nz), device="cuda", generator=gen)
    ph = 0.1 * torch.rand((ny, nz), device="cuda", generator=gen)
    return g, d, d / 20, torch.polar(1.0 + 0.1 * torch.rand((ny, nz), device="cuda", generator=gen), ph)


def gradient(M, g, d, b, probe, k, ws):
    f, ck = M.forward(g, d, b, probe, ckpt_every=k, ws=ws)
    M.workspace_status(ws)
    gd, gb, gp = M.adjoint(g, d, b, ck, k, 0.5 * f, ws=ws)
    M.workspace_status(ws)
    return [f, ck, gd, gb, gp]


@pytest.mark.parametrize("ny,nz,ns,k", [
    (16, 16, 9, 4), (16, 512, 12, 7), (512, 16, 11, 3), (32, 64, 33, 32), (64, 32, 40, 9), (64, 64, 5, 5),
    (64, 64, 6, 1), (128, 128, 70, 64), (128, 256, 37, 8), (256, 64, 21, 6), (256, 256, 66, 32), (256, 512, 19, 6),
    (512, 256, 18, 7), (512, 128, 14, 5), (512, 512, 40, 16), (512, 512, 7, 1), (16, 32, 200, 32)])
def test_bitwise_equal_to_per_pass(M, ny, nz, ns, k):
    g, d, b, probe = case(ny, nz, ns)
    M.set_schedule(1)
    ref = [x.clone() for x in gradient(M, g, d, b, probe, k, M.workspace(g, k))]
    M.set_schedule(0)
    ws = M.workspace(g, k)
    ws.view(torch.uint8).fill_(0xFF)   # nothing may depend on what a new workspace holds
    for _ in range(2):
        for r, o in zip(ref, gradient(M, g, d, b, probe, k, ws)):
            assert torch.equal(r, o)


def test_concurrent_calls(M):
    # calls of several host threads on streams of their own, each on its own workspace
    cases = [case(ny, nz, 60, seed=i) for i, (ny, nz) in enumerate([(512, 512), (256, 256), (512, 256), (64, 64)])]
    M.set_schedule(1)
    ref = [gradient(M, *c, 16, M.workspace(c[0], 16)) for c in cases]
    M.set_schedule(0)
    wss = [M.workspace(c[0], 16) for c in cases]
    torch.cuda.synchronize()
    out = [None] * len(cases)

    def run(i):
        with torch.cuda.stream(torch.cuda.Stream()):
            for _ in range(3):
                out[i] = gradient(M, *cases[i], 16, wss[i])
            torch.cuda.current_stream().synchronize()

    th = [threading.Thread(target=run, args=(i,)) for i in range(len(cases))]
    for t in th:
        t.start()
    for t in th:
        t.join()
    for r, o in zip(ref, out):
        for x, y in zip(r, o):
            assert torch.equal(x, y)


def test_captured_graph_replays(M):
    g, d, b, probe = case(128, 64, 50)
    ws = M.workspace(g, 0)
    out = torch.empty((128, 64), dtype=torch.complex64, device="cuda")
    M.forward(g, d, b, probe, ws=ws, out=out)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        M.forward(g, d, b, probe, ws=ws, out=out)
    for _ in range(3):
        d.mul_(0.9)
        M.set_schedule(1)
        ref, _ = M.forward(g, d, b, probe)
        M.set_schedule(0)
        torch.cuda.synchronize()
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(ref, out)


def test_wait_that_gives_up_is_reported(M):
    # spin limit 0: a wavefront that finds its input not yet there gives up at once; every kernel
    # still ends, the status reports it and the result is NaN; the next call is valid again
    g, d, b, probe = case(256, 256, 40)
    ws = M.workspace(g, 0)
    prev = M.set_barrier_spin_limit(0)
    try:
        f, _ = M.forward(g, d, b, probe, ws=ws)
        with pytest.raises(M.MslError) as e:
            M.workspace_status(ws)
        assert e.value.status == M.ERR_HIP
        assert torch.isnan(torch.view_as_real(f)).all()
    finally:
        M.set_barrier_spin_limit(prev)
    f, _ = M.forward(g, d, b, probe, ws=ws)
    M.workspace_status(ws)
    M.set_schedule(1)
    ref, _ = M.forward(g, d, b, probe)
    assert torch.equal(f, ref)


def test_payload_nans_do_not_stall(M):
    # a probe element with the exchange fields' own sentinel pattern
    g, d, b, probe = case(64, 64, 12)
    p = torch.view_as_real(probe)
    p.view(torch.int32)[3, 5, 0] = np.array([0xFFB5A3C7], np.uint32).view(np.int32)[0].item()
    ws = M.workspace(g, 0)
    f, _ = M.forward(g, d, b, probe, ws=ws)
    M.workspace_status(ws)
    assert torch.isnan(torch.view_as_real(f)).all()

"""A dataflow launch that gives up waiting (spin limit 0, set from the host: a wavefront that finds its
input not yet there gives up at once, and every kernel still ends): no output of the call may pass
for valid, also where it was complete before the wait or does not depend on it."""
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
    prev = msl.set_barrier_spin_limit(0)
    yield msl
    msl.set_barrier_spin_limit(prev)


def case(exact, ny=256, nz=128, ns=40):
    g = synth.Geometry(ny, nz, ns, 1.0, 1.0, 5.0, 0.1, math.radians(0.25), exact)
    gen = torch.Generator(device="cuda").manual_seed(3)
    d = 3e-5 * torch.rand((ns, ny, nz), device="cuda", generator=gen)
    return g, d, d / 20


def all_nan(*ts):
    return all(bool(torch.isnan(torch.view_as_real(t) if t.is_complex() else t).all()) for t in ts)


@pytest.mark.parametrize("exact", [0, 1])
def test_forward_outputs(M, exact):
    g, d, b = case(exact)
    ws = M.workspace(g, 8)
    f, ck = M.forward(g, d, b, ckpt_every=8, ws=ws)
    with pytest.raises(M.MslError):
        M.workspace_status(ws)
    assert all_nan(f, ck)


@pytest.mark.parametrize("k", [1, 8, 40])
@pytest.mark.parametrize("exact", [0, 1])
def test_gradients(M, exact, k):
    g, d, b = case(exact)
    ws = M.workspace(g, k)
    zero = M.set_barrier_spin_limit(1 << 22)
    f, ck = M.forward(g, d, b, ckpt_every=k, ws=ws)
    M.workspace_status(ws)
    M.set_barrier_spin_limit(zero)
    out = M.adjoint(g, d, b, ck, k, f, ws=ws)
    with pytest.raises(M.MslError):
        M.workspace_status(ws)
    assert all_nan(*out)
    assert not all_nan(f) and not all_nan(ck)   # the inputs stay


def test_noalloc_outputs(M):
    g, d, b = case(0)
    f, ck = M.forward_noalloc(g, d, b, ckpt_every=8)
    assert all_nan(f, ck)


def test_noalloc_status(M):
    g, d, b = case(0)
    M.forward_noalloc(g, d, b)
    with pytest.raises(M.MslError) as e:
        M.noalloc_status()
    assert e.value.status == M.ERR_HIP
    zero = M.set_barrier_spin_limit(1 << 22)
    for ny, nz, exact in ((256, 128, 0), (1024, 1024, 0), (512, 512, 1)):   # with a dataflow launch and without
        M.forward_noalloc(*case(exact, ny, nz, 6))
        M.noalloc_status()
    M.set_barrier_spin_limit(zero)


@pytest.mark.parametrize("graphs", [False, True])
@pytest.mark.parametrize("where", ["forward", "adjoint"])
def test_reconstruction_raises_and_keeps_theta(M, where, graphs):
    # a sweep that gives up is reported where the driver waits for the GPU, and its gradients never
    # reach theta; with the limit restored the same driver goes on
    import numpy as np
    from paper_2212_01253_amd import recon
    region = {"s0": 0, "ns": 40, "y0": 16, "ny": 16, "z0": 0, "nz": 64, "beta_over_delta": 0.05}
    g, d, b = case(0, 64, 64)
    zero = M.set_barrier_spin_limit(1 << 22)
    R = recon.Reconstructor(g, d.cpu().numpy(), b.cpu().numpy(), region, np.full((64, 64), 10.0), 1.0, ckpt_every=8,
                            graphs=graphs)
    theta = np.full((40, 16, 64), 1e-5, np.float32)
    full = R.run(theta, 3).losses
    R.set_theta(theta)
    step = R._run

    def failing(which):
        # captured launches keep the limit they were captured with: the call that fails is run eagerly
        if which == ("loss" if where == "forward" else "adjoint") and R.t >= 1:
            M.set_barrier_spin_limit(0)
            (R._loss_calls if which == "loss" else R._adjoint_calls)()
            M.set_barrier_spin_limit(1 << 22)
        else:
            step(which)

    R._run = failing
    with pytest.raises(M.MslError) as e:
        R.run(theta, 3)
    assert e.value.status == M.ERR_HIP and R.t == 1
    assert bool(torch.isfinite(R.theta).all()) and bool(torch.isfinite(R.m).all())
    R._run = step
    assert R.run(theta, 3).losses == full
    M.set_barrier_spin_limit(zero)

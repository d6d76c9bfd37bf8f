"""Which launch shapes leave the dataflow schedule in place: any number of lines per workgroup (it has its
own), and the points per lane its kernels have, set or default; other points per lane run per pass.
Whether a call made a dataflow launch shows at spin limit 0 (set from the host: its waits give up at
once, every kernel ends), where only such a launch can fail.  Results are compared bit for bit.
Calls of few passes, which such a launch would only slow down, run per pass."""
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
    before = msl.get_tuning()
    yield msl
    msl.set_schedule(0)
    msl.restore_tuning(before)


def forward_fails(M, g, d, ws):
    prev = M.set_barrier_spin_limit(0)
    try:
        M.forward(g, d, d / 20, ws=ws)
        M.workspace_status(ws)
        return False
    except M.MslError:
        return True
    finally:
        M.set_barrier_spin_limit(prev)


@pytest.mark.parametrize("exact,ns,flow", [(0, 5, False), (0, 6, False), (0, 8, True), (1, 3, False), (1, 5, True)])
def test_short_calls(M, exact, ns, flow):
    g = synth.Geometry(256, 256, ns, 1.0, 1.0, 5.0, 0.1, math.radians(0.25), exact)
    d = 3e-5 * torch.rand((ns, 256, 256), device="cuda")
    assert forward_fails(M, g, d, M.workspace(g, 0)) == flow


@pytest.mark.parametrize("lines,points,flow", [
    ({}, {}, True), ({256: 1, 128: 4}, {}, True), ({256: 4}, {256: 4, 128: 4}, True), ({}, {256: 4}, True),
    ({}, {256: 8}, False), ({128: 2}, {128: 8}, False), ({512: 2, 64: 16}, {512: 4}, True)])
def test_shapes(M, lines, points, flow):
    g = synth.Geometry(256, 128, 40, 1.0, 1.0, 5.0, 0.1, math.radians(0.25), 0)
    gen = torch.Generator(device="cuda").manual_seed(3)
    d = 3e-5 * torch.rand((40, 256, 128), device="cuda", generator=gen)
    M.set_tuning(lines, points_per_lane=points)
    ws = M.workspace(g, 0)
    M.set_schedule(1)
    ref, _ = M.forward(g, d, d / 20, ws=ws)
    M.set_schedule(0)
    f, _ = M.forward(g, d, d / 20, ws=ws)
    assert torch.equal(f, ref)
    assert forward_fails(M, g, d, ws) == flow


MASKED = """
import math, torch
from paper_2212_01253_amd import msl, synth
g = synth.Geometry(256, 128, 40, 1.0, 1.0, 5.0, 0.1, math.radians(0.25), 0)
d = 3e-5 * torch.rand((40, 256, 128), device="cuda")
ws = msl.workspace(g, 0)
msl.set_barrier_spin_limit(0)
msl.forward(g, d, d / 20, ws=ws)
msl.workspace_status(ws)
print("per pass")
"""


def test_process_wide_mask(M):
    # a process whose queues are masked by the environment runs per pass (the mask here leaves every unit in)
    import os
    import subprocess
    import sys
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    n = torch.cuda.get_device_properties(0).multi_processor_count
    r = subprocess.run([sys.executable, "-c", MASKED], cwd=root, env={**os.environ, "HSA_CU_MASK": f"0:0-{n - 1}"},
                       capture_output=True, text=True, timeout=110)
    assert r.returncode == 0 and r.stdout.strip() == "per pass", r.stdout + r.stderr

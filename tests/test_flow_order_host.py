"""Host-only check of the dataflow schedule's ordering (CPU): builds and runs csrc/flow_check.cpp.

The launch hands the field from pass to pass without barriers, so what orders the resets of
an exchange field against its next elements and its next readers is worth a proof: the check
follows every wavefront's knowledge through the passes of all 36 grids.  Resets behind a
pass's output are not enough where the axes have different numbers of workgroups (one axis of 512 points,
the other shorter), which the check has to find.
"""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = os.path.join(ROOT, "paper_2212_01253_amd", "csrc", "flow_check.cpp")


@pytest.fixture(scope="module")
def check(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    exe = str(tmp_path_factory.mktemp("flow") / "flow_check")
    subprocess.run([hipcc, "--offload-host-only", "-std=c++17", "-O2", "-I", os.path.join(ROOT, "include"),
                    "-o", exe, SRC], check=True, capture_output=True)
    return lambda *a: subprocess.run([exe, *a], capture_output=True, text=True, timeout=300)


def test_every_grid_is_ordered(check):
    r = check()
    assert r.returncode == 0 and r.stdout.strip() == "OK", r.stdout + r.stderr


def test_resets_behind_the_output_are_found_wanting(check):
    r = check("late")
    short = (16, 32, 64, 128, 256)
    assert r.returncode == 1
    assert {l.split(":")[0] for l in r.stdout.splitlines()} == {f"{a} x {b}" for n in short for a, b in ((n, 512), (512, n))}

"""Build libmsl.so for gfx950 with hipcc (in-tree, next to this file)."""
from __future__ import annotations

import os
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
SRCS = [os.path.join(HERE, "csrc", f) for f in ("msl.hip", "msl_flow.hip", "msl_flow_fwd.hip", "msl_flow_rev.hip", "msl_flow_stack.hip",
                                                 "msl_flow_xfwd.hip", "msl_flow_xrev.hip", "msl_recon.hip", "msl_nn.hip")]
OUT = os.path.join(HERE, "libmsl.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

FLAGS = [
    "-O3", "--offload-arch=gfx950", "-std=c++17", "-fPIC",
    # no implicit multiply-add contraction: the kernels place every FMA explicitly
    "-ffp-contract=off",
    # keep the compiler from emitting packed FP32 instructions
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-I" + os.path.join(ROOT, "include"),
]


def build(verbose: bool = True) -> str:
    noise = "is not a recognized feature for this target"

    def run(cmd):
        r = subprocess.run(cmd, capture_output=True, text=True)
        out = "\n".join(l for l in (r.stdout + r.stderr).splitlines() if noise not in l and "(ignoring feature)" not in l)
        if r.returncode != 0:
            raise RuntimeError(f"hipcc failed ({r.returncode}):\n{' '.join(cmd)}\n{out}")
        return out

    tmp = OUT + ".tmp"
    with tempfile.TemporaryDirectory() as d:
        objs = [os.path.join(d, os.path.basename(s) + ".o") for s in SRCS]
        with ThreadPoolExecutor(len(SRCS)) as pool:   # the sources side by side, then one link
            outs = list(pool.map(lambda so: run([HIPCC, *FLAGS, "-c", "-o", so[1], so[0]]), zip(SRCS, objs)))
        outs.append(run([HIPCC, *FLAGS, "-shared", "-o", tmp, *objs]))
    err = "\n".join(o for o in outs if o)
    os.replace(tmp, OUT)
    if verbose and err.strip():
        print(err, file=sys.stderr)
    return OUT


if __name__ == "__main__":
    print(build())

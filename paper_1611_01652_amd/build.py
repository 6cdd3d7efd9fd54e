"""Build the HIP library libsim_hip.so for gfx950 (in-tree)."""
from __future__ import annotations

import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
OUT = os.path.join(HERE, "libsim_hip.so")

# (source, extra flags): the per-env kernels are compiled once per team width,
# all at once
SOURCES = [("team_kernels.hip", [f"-DSIM_TEAM={t}"]) for t in (64, 32, 16, 8, 4, 2, 1)] + [
    (s, []) for s in ("sim_kernels.hip", "wsn_kernels.hip", "render_kernels.hip", "sim_api.cpp", "model_pack.cpp")]

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # no packed FP32 instructions (v_pk_*_f32) are emitted
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-variable", "-Wno-unused-but-set-variable",
]


def build(verbose: bool = False) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    bdir = os.path.join(HERE, "_build")
    os.makedirs(bdir, exist_ok=True)
    cmds, objs = [], []
    for src, extra in SOURCES:
        obj = os.path.join(bdir, src + "".join(extra) + ".o")
        cmds.append([hipcc] + HIPCC_FLAGS + extra + ["-x", "hip", "-I", os.path.join(ROOT, "include"), "-c",
                                             os.path.join(CSRC, src), "-o", obj])
        objs.append(obj)
    # the translation units are independent: compile them at once
    procs = []
    for cmd in cmds:
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append(subprocess.Popen(cmd))
    failed = [c for c, p in zip(cmds, procs) if p.wait() != 0]
    if failed:
        raise subprocess.CalledProcessError(1, failed[0])
    tmp = OUT + ".tmp"
    cmd = [hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp] + objs
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    os.replace(tmp, OUT)
    return OUT


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))

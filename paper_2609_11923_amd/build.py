"""Build libcfr.so in place with hipcc for gfx950 (host compile; no GPU needed).

    python -m paper_2609_11923_amd.build
"""
from __future__ import annotations

import os
import shutil
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
SO = os.path.join(HERE, "libcfr.so")
SOURCES = ["compiler.cpp", "kernels.hip", "evaluate.hip", "runtime.hip", "mlp.hip"]
PARTS = {"kernels.hip": 5}   # compiled once per CFR_PART, side by side
ARCH = "gfx950"


def hipcc() -> str:
    for c in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", shutil.which("hipcc")):
        if c and os.path.exists(c):
            return c
    raise RuntimeError("hipcc not found")


def flags() -> list[str]:
    return [
        f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC", "-shared", "-Wall",
        # packed FP32 instructions stay off in every kernel
        "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
        "-I", os.path.join(HERE, "..", "include"),
    ]


def build(verbose: bool = False) -> str:
    """Always recompiles (callers decide when a build is needed)."""
    objs = []
    tmpdir = os.path.join(HERE, "_build")
    os.makedirs(tmpdir, exist_ok=True)
    cc = hipcc()
    procs = []
    for src, part in [(s, p) for s in SOURCES for p in range(PARTS.get(s, 1))]:
        obj = os.path.join(tmpdir, f"{src}.{part}.o")
        cmd = [cc] + [f for f in flags() if f != "-shared"] + ["-c", os.path.join(CSRC, src), "-o", obj]
        if src in PARTS:
            cmd.append(f"-DCFR_PART={part}")
        if src.endswith(".cpp"):
            cmd = [cc, "-O3", "-std=c++17", "-fPIC", "-Wall", "-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT), src))
        objs.append(obj)
    for p, src in procs:
        out, _ = p.communicate()
        text = out.decode(errors="replace")
        # the host pass warns that it does not know the packed-fp32 feature flag; that is expected
        lines = [ln for ln in text.splitlines() if "packed-fp32-ops" not in ln and ln.strip()]
        if p.returncode != 0:
            raise RuntimeError(f"hipcc failed on {src}:\n{text}")
        if verbose and lines:
            print("\n".join(lines))
    tmp = SO + ".tmp"
    cmd = [cc, f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", tmp] + objs
    subprocess.check_call(cmd)
    os.replace(tmp, SO)
    return SO


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))

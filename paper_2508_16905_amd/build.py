"""Build the HIP library for gfx950 in-tree (``libtriaccel.so`` next to this file)."""

from __future__ import annotations

import os
import subprocess
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libtriaccel.so")
SOURCES = ["kernels.hip", "update.hip", "update_local.hip", "update_resize.hip", "power.hip", "api.hip"]

HIPCC_FLAGS = [
    "--offload-arch=gfx950",
    "-O3",
    "-std=c++17",
    "-fPIC",
    "-shared",
    # every fused multiply-add in the kernels is written as fmaf(); nothing else may be contracted
    "-ffp-contract=off",
    "-fno-fast-math",
    "-fno-gpu-flush-denormals-to-zero",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # a kernel's leading pointer arguments are in scalar registers when its wavefronts start, instead of one memory
    # latency later (EfficientNet-B0 set, 16 bits, without a probe: 15.4 -> 14.8 us a step; 41 tensors of 1.0 M with a
    # probe 22.9 -> 22.0)
    "-mllvm", "-amdgpu-kernarg-preload-count=16",
    "-Wall",
    "-Wno-unused-function",
]


def build_library(force: bool = True, verbose: bool = False) -> str:
    srcs = [os.path.join(CSRC, s) for s in SOURCES]
    deps = srcs + [os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith(".h")]
    deps.append(os.path.join(os.path.dirname(HERE), "include", "triaccel.h"))
    if not force and os.path.exists(LIB) and all(os.path.getmtime(LIB) >= os.path.getmtime(d) for d in deps):
        return LIB
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    flags = [f for f in HIPCC_FLAGS if f != "-shared"]
    # the translation units are compiled side by side (the kernels dominate), then linked
    with tempfile.TemporaryDirectory(prefix="triaccel_build_") as tmp:
        objs, procs = [], []
        for src in srcs:
            obj = os.path.join(tmp, os.path.basename(src) + ".o")
            cmd = [hipcc] + flags + ["-c", src, "-o", obj]
            if verbose:
                print(" ".join(cmd))
            procs.append((cmd, subprocess.Popen(cmd)))
            objs.append(obj)
        for cmd, proc in procs:
            if proc.wait() != 0:
                for _, other in procs:
                    other.wait()
                raise subprocess.CalledProcessError(proc.returncode, cmd)
        link = [hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB] + objs
        if verbose:
            print(" ".join(link))
        subprocess.run(link, check=True)
    return LIB


if __name__ == "__main__":
    print(build_library(force=True, verbose=True))

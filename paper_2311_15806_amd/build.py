"""Builds libpipe_hip.so (the C-ABI library) for gfx950 with hipcc, in-tree."""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libpipe_hip.so")
OBJ_DIR = os.path.join(HERE, "_build")

# (source, extra flags).  The files whose fp32 results feed rounding decisions are built
# with floating-point contraction off.
# Kernels of a few microseconds get their scalar arguments in registers with the launch, instead of loading them from
# host memory first: 0.15 us of a launch (1000 x 768 affine codes, 32 x 256 x 14 x 14 and 32 x 384 x 28 x 28 images, calls of 20 to 29 us -0.9 %).
PRELOAD = ["-mllvm", "-amdgpu-kernarg-preload-count=16"]
SOURCES = [
    ("pipe_api.hip", []),
    ("pipe_expand.hip", ["-ffp-contract=off"]),
    ("pipe_quant.hip", ["-ffp-contract=off"] + PRELOAD),
    ("pipe_gemm.hip", []),
    ("pipe_gemm_bins.hip", PRELOAD),
    ("pipe_gemv.hip", PRELOAD),
    ("pipe_resident.hip", []),
    ("pipe_probe.hip", []),
    ("pipe_diag.hip", ["-ffp-contract=off"]),
    ("pipe_depthwise.hip", ["-ffp-contract=off"] + PRELOAD),
]

COMMON = [
    "-O3", "-std=c++17", "--offload-arch=gfx950", "-fPIC",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function", "-Wno-unknown-warning-option",
]


def _hipcc() -> str:
    for c in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if c and (os.path.isabs(c) and os.path.exists(c) or not os.path.isabs(c)):
            return c
    return "hipcc"


def _compile(src: str, extra) -> str:
    obj = os.path.join(OBJ_DIR, os.path.splitext(src)[0] + ".o")
    cmd = [_hipcc()] + COMMON + list(extra) + ["-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    out = "\n".join(l for l in (r.stdout + r.stderr).splitlines()
                    if "packed-fp32-ops" not in l)      # the host pass does not know the feature
    if r.returncode != 0:
        raise RuntimeError("hipcc failed for %s:\n%s" % (src, out))
    if out.strip():
        sys.stderr.write(out + "\n")
    return obj


def build_library(verbose: bool = True) -> str:
    os.makedirs(OBJ_DIR, exist_ok=True)
    srcs = [(s, f) for s, f in SOURCES if os.path.exists(os.path.join(CSRC, s))]
    with ThreadPoolExecutor(max_workers=min(8, len(srcs))) as ex:
        objs = list(ex.map(lambda sf: _compile(*sf), srcs))
    cmd = [_hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB] + objs
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n" + r.stdout + r.stderr)
    if verbose:
        print("built", LIB)
    return LIB


if __name__ == "__main__":
    build_library()

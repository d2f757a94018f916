"""Build libeqb.so for gfx950 with hipcc, in place next to this file.

    python -m paper_2609_28053_amd.build          # or: python paper_2609_28053_amd/build.py
"""
from __future__ import annotations

import concurrent.futures
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
SOURCES = [os.path.join(CSRC, f) for f in ("eqb_api.hip", "margin.hip", "select.hip", "balance.hip", "variants.hip",
                                          "layer_noalloc.hip")]
# The routing kernels are compiled on their own (one object per expert count,
# in parallel: every fan-out has its own unrolled kernel), without IEEE mode: their
# float maxima and medians then need no NaN quieting, which lets the compiler
# fold each DPP group maximum into one instruction and schedule around its
# wait states.  Their operands are keys and finite scores, never NaN (finite
# inputs are a precondition of the library).
ROUTE_SOURCE = os.path.join(CSRC, "route.hip")
ROUTE_EXPERTS = (256, 128, 64, 32, 16, 8)
ROUTE_FLAGS = ["-mno-amdgpu-ieee", "-fno-honor-nans"]
OUT = os.path.join(HERE, "libeqb.so")
ARCH = os.environ.get("EQB_OFFLOAD_ARCH", "gfx950")

FLAGS = [
    f"--offload-arch={ARCH}",
    "-O3",
    "-std=c++17",
    "-fPIC",
    "-shared",
    "-ffp-contract=off",               # no fused multiply-add anywhere on the path
    # packed FP32 instructions are kept out of the generated code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall",
]


# hipcc hands -Xclang options to the host (x86) pass as well, which reports
# the GPU-only feature as unknown and ignores it; -Xclang cannot be restricted
# to the device pass (-Xarch_device does not forward it).  The device pass
# applies it: tests/test_build.py disassembles the built library's gfx950 code
# and finds no packed FP32 instruction.  That one known line is dropped from
# the build log; anything else the compiler prints is shown.
_HOST_FEATURE_NOTE = "'-packed-fp32-ops' is not a recognized feature for this target (ignoring feature)"


def _run(cmd, verbose):
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    err = "".join(l for l in res.stderr.splitlines(keepends=True) if l.strip() != _HOST_FEATURE_NOTE)
    if res.returncode != 0:
        sys.stderr.write(res.stdout + err)
        raise RuntimeError(f"hipcc failed with status {res.returncode}")
    if verbose and err:
        sys.stderr.write(err)


# Host-side sanitizers for the C ABI shim (argument checks, partition
# tables, workspace carving): AddressSanitizer and UndefinedBehaviorSanitizer
# on the host pass only.  The GPU code is built as usual; the result is a
# separate library for CPU-only test runs (tests/test_abi_sanitized.py).
SANITIZE_FLAGS = ["-Xarch_host", "-fsanitize=address", "-Xarch_host", "-fsanitize=undefined",
                  "-Xarch_host", "-fno-omit-frame-pointer", "-Xarch_host", "-fno-sanitize-recover=all"]


def build(verbose: bool = False, extra=(), out: str = OUT, sanitize: bool = False) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    extra = list(extra) + (SANITIZE_FLAGS if sanitize else [])
    tmp = out + ".tmp"
    inc = ["-I", os.path.join(ROOT, "include"), "-I", CSRC]
    compile_flags = [f for f in FLAGS if f != "-shared"]
    jobs = [([*compile_flags, *ROUTE_FLAGS, f"-DEQB_ROUTE_E={e}"], ROUTE_SOURCE, f"{out}.route{e}.o")
            for e in ROUTE_EXPERTS]
    jobs += [(compile_flags, src, f"{out}.{os.path.basename(src)}.o") for src in SOURCES]
    objs = [obj for _, _, obj in jobs]
    try:
        with concurrent.futures.ThreadPoolExecutor(min(8, os.cpu_count() or 1)) as pool:
            for f in [pool.submit(_run, [hipcc, *flags, *extra, *inc, "-c", src, "-o", obj], verbose)
                      for flags, src, obj in jobs]:
                f.result()
        _run([hipcc, *FLAGS, *extra, *objs, "-o", tmp], verbose)
    finally:
        for obj in objs:
            if os.path.exists(obj):
                os.remove(obj)
    os.replace(tmp, out)
    return out


if __name__ == "__main__":
    print(build(verbose=True, extra=sys.argv[1:]))

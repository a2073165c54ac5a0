"""Build libfrbx.so in-tree with hipcc for gfx950.

    python -m paper_1801_02391_amd.build

Compiles the HIP kernels and the host side of the library and links them
into paper_1801_02391_amd/libfrbx.so.  Every build recompiles from source.
"""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
BUILD = os.path.join(ROOT, "_build")
LIB = os.path.join(PKG, "libfrbx.so")

ARCH = "gfx950"
# Packed FP32 instructions are kept out of every device code object.
DEVICE_FLAGS = ["-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]
# Matrix-core results go straight to VGPRs (no accumulator read-back).
KERNEL_FLAGS = ["-mllvm", "-amdgpu-mfma-vgpr-form=true"]
COMMON = ["-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function", "-Wno-unused-variable",
          f"--offload-arch={ARCH}"]


RTC_SOURCE = os.path.join(CSRC, "frbx_rtc_source.inc")


def write_rtc_source() -> str:
    """Write csrc/frbx_rtc_source.inc: the float32 fringe kernel's device
    code (frbx_internal.h + frbx_fringe.h) as a C++ raw string, for the
    library to compile kernels specialised to an IF lattice with hipRTC."""
    parts = []
    for name in ("frbx_internal.h", "frbx_fringe.h"):
        for line in open(os.path.join(CSRC, name)):
            if line.strip() in ('#include "frbx_internal.h"', "#pragma once"):
                continue
            parts.append(line)
    text = "".join(parts)
    if ")FRBXRTC" in text:
        raise RuntimeError("raw-string delimiter found in the kernel source")
    out = ("// Generated by paper_1801_02391_amd/build.py from frbx_internal.h and\n"
           "// frbx_fringe.h: the device code compiled at run time by hipRTC.\n"
           'static const char kFringeRtcSource[] = R"FRBXRTC(' + text + ')FRBXRTC";\n')
    tmp = RTC_SOURCE + ".tmp"
    with open(tmp, "w") as f:
        f.write(out)
    os.replace(tmp, RTC_SOURCE)
    return RTC_SOURCE


def _hipcc():
    h = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(h):
        raise RuntimeError("hipcc not found")
    return h


def _run(cmd, verbose):
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        sys.stderr.write(r.stdout + r.stderr)
        raise RuntimeError(f"build step failed: {' '.join(cmd[:3])} ...")
    return r


def build(verbose: bool = True) -> str:
    os.makedirs(BUILD, exist_ok=True)
    hipcc = _hipcc()
    write_rtc_source()
    units = [("frbx_kernels.hip", ["-O3", *KERNEL_FLAGS]),
             ("frbx_screen.hip", ["-O3", *KERNEL_FLAGS]),
             ("frbx_jit.cpp", ["-O2"]),
             # float64 tables must not be contracted into FMAs: keep Eq. 2
             # rounding bit-identical to a plain evaluation of the formula
             ("frbx_host.cpp", ["-O2", "-ffp-contract=off"])]

    def compile_unit(unit):
        src, flags = unit
        obj = os.path.join(BUILD, os.path.splitext(src)[0] + ".o")
        _run([hipcc, "-c", *flags, *COMMON, *DEVICE_FLAGS, os.path.join(CSRC, src), "-o", obj], verbose)
        return obj

    with ThreadPoolExecutor(len(units)) as pool:
        objs = list(pool.map(compile_unit, units))
    tmp = LIB + ".tmp"
    _run([hipcc, "-shared", f"--offload-arch={ARCH}", "-fPIC", *objs, "-lhiprtc", "-o", tmp], verbose)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    build(verbose="-q" not in sys.argv)
    print(LIB)

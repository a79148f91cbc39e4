"""Build libamap.so (HIP kernels + host composer + C ABI) for gfx950 with hipcc, and the binding's native part with gcc."""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
import sysconfig

_HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(_HERE)
CSRC = os.path.join(_HERE, "csrc")
LIB = os.path.join(_HERE, "libamap.so")
# CPython extension, from a Python call to the library: its name holds the interpreter's ABI, and another one looks for another name
CALL = os.path.join(_HERE, "_amap_call" + sysconfig.get_config_var("EXT_SUFFIX"))

SOURCES = ["amap_compose.cpp", "amap_graph.cpp", "amap_layout.cpp", "amap_host.cpp", "amap_plan.cpp", "amap_plan_check.cpp", "amap_kernels.hip",
           "amap_gemm.hip", "amap_gemm_ring.hip"]

FLAGS = [
    "-O3", "-std=c++17", "-fPIC", "-shared", "--offload-arch=gfx950",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wextra", "-Wno-unused-command-line-argument",
    # The piece kernel reads its by-value argument block through many inlined
    # bodies.  Past a fixed number of uses the optimiser stops reading the
    # block in place and copies all of it to private memory (3 KB of scratch
    # per lane, every field access a scratch load); lift that limit.
    "-mllvm", "-instcombine-max-copied-from-constant-users=100000",
    "-Rpass-analysis=kernel-resource-usage",
]


def build_lib(verbose: bool = False, extra=()) -> str:
    cmd = ["hipcc", *FLAGS, *extra, "-I", os.path.join(ROOT, "include"), "-I", CSRC]
    for s in SOURCES:
        path = os.path.join(CSRC, s)
        cmd += (["-x", "hip", path] if s.endswith(".hip") else ["-x", "c++", path])
    cmd += ["-o", LIB]
    if verbose:
        print(" ".join(cmd), file=sys.stderr)
    # the host pass of hipcc prints one harmless "not a recognized feature"
    # line per function for the packed-fp32 switch; drop those, keep the rest
    r = subprocess.run(cmd, stderr=subprocess.PIPE, text=True)
    usage = kernel_usage(r.stderr)
    after_remark = False
    for line in r.stderr.splitlines():
        if "packed-fp32-ops' is not a recognized feature" in line:
            continue
        if "kernel-resource-usage" in line:
            after_remark = True
            continue
        if after_remark and line.split("|")[0].strip().isdigit() or (after_remark and line.strip().startswith("|")):
            continue  # the source excerpt under a remark
        after_remark = False
        print(line, file=sys.stderr)
    if r.returncode != 0:
        raise subprocess.CalledProcessError(r.returncode, cmd)
    if verbose:
        for name, u in usage.items():
            print(f"{name}: {u}", file=sys.stderr)
    wrong = check_usage(usage)
    if wrong:
        os.remove(LIB)
        raise RuntimeError("; ".join(wrong))
    build_call()
    return LIB


def build_call():
    """The extension's path, or None where it cannot be built: the binding does without."""
    include = sysconfig.get_path("include")
    lacks = "gcc" if not shutil.which("gcc") else "Python.h" if not os.path.exists(os.path.join(include, "Python.h")) else None
    if lacks:
        if os.path.exists(CALL):
            os.remove(CALL)   # of another state of the source
        print(f"{CALL} not built (no {lacks}): Python calls go through ctypes", file=sys.stderr)
        return None
    subprocess.run(["gcc", "-O2", "-std=c99", "-fPIC", "-shared", "-Wall", "-Wextra", "-I", include,
                    os.path.join(CSRC, "amap_call.c"), "-o", CALL], check=True)
    untagged = os.path.join(_HERE, "_amap_call.so")   # built so before: any interpreter would load it
    if os.path.exists(untagged):
        os.remove(untagged)
    return CALL


# Wavefronts per SIMD of the map kernels.  They are bound by memory and every form inlined into amap_pieces_kernel shares its
# registers: 74 instead of 66 VGPRs for the sake of one form took it from 7 to 6 and the cross-lane form from 213 to 230 us
# ([8192,8,64,64] 2-byte elements to channels-last, 1.07 GB).
MIN_OCCUPANCY = {"amap_rows_kernel": 8, "amap_rows_few_kernel": 8, "amap_rows_multi_kernel": 8, "amap_tile16_kernel": 8, "amap_flat_kernel": 8,
                 "amap_pieces_kernelILi2E": 7, "amap_pieces_kernelILi4E": 6}


def check_usage(usage: dict) -> list:
    """What is wrong with the kernels' resource figures, one line per fault."""
    wrong = []
    for name, u in usage.items():
        if u.get("ScratchSize [bytes/lane]", 0) != 0:
            wrong.append(f"{name} uses scratch memory (argument block copied or registers spilled): {u}")
        # the GEMM kernels address their dynamic LDS from 0: a static allocation (an array the compiler moved there) would overlap it
        if "gemm" in name and u.get("LDS Size [bytes/block]", 0) != 0:
            wrong.append(f"{name} is a GEMM kernel with static LDS: {u}")
        for kernel, least in MIN_OCCUPANCY.items():
            if kernel in name and u.get("Occupancy [waves/SIMD]", least) < least:
                wrong.append(f"{name} keeps fewer than {least} wavefronts per SIMD: {u}")
    return wrong


def kernel_usage(stderr: str) -> dict:
    """Per-kernel register / scratch figures from the compiler's resource remarks."""
    usage, cur = {}, None
    for line in stderr.splitlines():
        if "remark:" not in line:
            continue
        body = line.split("remark:", 1)[1].split("[-Rpass-analysis")[0].strip()
        if body.startswith("Function Name:"):
            cur = usage.setdefault(body.split(":", 1)[1].strip(), {})
        elif cur is not None and ":" in body:
            k, v = body.rsplit(":", 1)
            try:
                cur[k.strip()] = int(v)
            except ValueError:
                pass
    return usage


if __name__ == "__main__":
    print(build_lib(verbose=True))

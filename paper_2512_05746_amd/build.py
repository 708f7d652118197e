"""Builds libhq.so (the C-ABI HIP library) in-tree for gfx950 with hipcc."""
from __future__ import annotations

import os
import subprocess
import sys

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
LIB = os.path.join(PKG, "libhq.so")
SOURCES = ["hq_hadamard_quant.hip", "hq_int_gemm.hip", "hq_int_gemm_128x128.hip",
           "hq_int_gemm_64x128.hip", "hq_int_gemm_64x64.hip", "hq_conv3x3_wave.hip", "hq_conv3x3_res.hip", "hq_conv3x3_fused.hip", "hq_resident.hip", "hq_resident_pertap.hip", "hq_resident_sum.hip", "hq_resident_linear.hip", "hq_linear_fused.hip", "hq_int_gemm_anyk.hip",
           "hq_single_weights.hip", "hq_width_quant.hip"]
HEADERS = ["hq_common.h", "hq_int_gemm_kernel.h", "hq_hadamard_mfma.h", "hq_conv3x3_res_kernel.h", "hq_resident_kernel.h", "hq_fp6.h"]

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # hipcc -O3 otherwise forms packed-fp32 instructions from ordinary float code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # keep MFMA results in ordinary vector registers (no copies out of the accumulation file)
    "-mllvm", "-amdgpu-mfma-vgpr-form=1",
    "-Wall", "-Wno-unused-function",
]


def sources():
    return [os.path.join(CSRC, s) for s in SOURCES]


def is_stale() -> bool:
    if not os.path.exists(LIB):
        return True
    t = os.path.getmtime(LIB)
    deps = sources() + [os.path.join(CSRC, h) for h in HEADERS] + [os.path.join(ROOT, "include", "hq.h")]
    return any(os.path.getmtime(d) > t for d in deps)


def _run(cmd, verbose):
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    out = "\n".join(l for l in res.stdout.splitlines() if "packed-fp32-ops" not in l)
    if res.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + out)
    if verbose and out.strip():
        print(out)


def build_lib(verbose: bool = False) -> str:
    """Compiles every source to an object (in parallel) and links libhq.so."""
    from concurrent.futures import ThreadPoolExecutor

    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    objdir = os.path.join(PKG, "_build")
    os.makedirs(objdir, exist_ok=True)
    inc = ["-I", os.path.join(ROOT, "include"), "-I", CSRC]
    objs = [os.path.join(objdir, os.path.basename(s) + ".%d.o" % os.getpid()) for s in sources()]
    jobs = [[hipcc] + HIPCC_FLAGS + inc + ["-c", src, "-o", obj] for src, obj in zip(sources(), objs)]
    with ThreadPoolExecutor(max_workers=min(8, len(jobs))) as pool:
        list(pool.map(lambda c: _run(c, verbose), jobs))
    tmp = LIB + ".tmp%d" % os.getpid()
    _run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp] + objs, verbose)
    for o in objs:
        os.remove(o)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build_lib(verbose=True))

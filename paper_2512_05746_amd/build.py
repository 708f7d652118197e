"""Builds libhq.so (the C-ABI HIP library) in-tree for gfx950 with hipcc, and the native part of its Python face
(_marshal.so, host code only) with g++."""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
LIB = os.path.join(PKG, "libhq.so")
MARSHAL = os.path.join(PKG, "_marshal.so")
MARSHAL_SOURCE = os.path.join(CSRC, "marshal.cpp")
SOURCES = ["hq_hadamard_quant.hip", "hq_int_gemm.hip", "hq_int_gemm_128x128.hip",
           "hq_int_gemm_64x128.hip", "hq_int_gemm_64x64.hip", "hq_conv3x3_wave.hip", "hq_conv3x3_fused.hip",
           "hq_resident.hip", "hq_resident_pertap.hip", "hq_resident_wholetaps.hip",
           "hq_resident_wholetaps_ragged.hip", "hq_resident_sum.hip", "hq_resident_sum_ragged.hip",
           "hq_resident_planes.hip", "hq_resident_bytes.hip", "hq_linear_fp6.hip", "hq_linear_fused.hip",
           "hq_int_gemm_anyk.hip",
           "hq_single_weights.hip", "hq_width_quant.hip"]
HEADERS = ["hq_common.h", "hq_int_gemm_kernel.h", "hq_hadamard_mfma.h", "hq_conv3x3_res_kernel.h",
           "hq_resident_kernel.h", "hq_fp6.h", "hq_buffer.h"]

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


def built_for() -> str:
    """The interpreter and the PyTorch whose interfaces _marshal.so is compiled against; the file holds this text."""
    import torch
    return "built for Python %s, PyTorch %s" % (sys.version.split()[0], torch.__version__)


def _marshal_matches() -> bool:
    with open(MARSHAL, "rb") as f:
        return built_for().encode() in f.read()


def is_stale() -> bool:
    abi = os.path.join(ROOT, "include", "hq.h")
    deps = {LIB: sources() + [os.path.join(CSRC, h) for h in HEADERS] + [abi], MARSHAL: [MARSHAL_SOURCE, abi]}
    return any(not os.path.exists(out) or any(os.path.getmtime(d) > os.path.getmtime(out) for d in ds)
               for out, ds in deps.items()) or not _marshal_matches()


def _run(cmd, verbose):
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    out = "\n".join(l for l in res.stdout.splitlines() if "packed-fp32-ops" not in l)
    if res.returncode != 0:
        raise RuntimeError("%s failed:\n%s" % (os.path.basename(cmd[0]), out))
    if verbose and out.strip():
        print(out)


def marshal_command(out: str):
    """The g++ command of _marshal.so: PyTorch's headers and libraries, no device code."""
    import torch
    torch_dir = os.path.dirname(torch.__file__)
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
           "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI), '-DHQ_BUILT_FOR="%s"' % built_for(),
           "-I", os.path.join(ROOT, "include")]
    for d in (os.path.join(torch_dir, "include"), os.path.join(torch_dir, "include", "torch", "csrc", "api", "include"),
              os.path.join(rocm, "include"), sysconfig.get_paths()["include"]):
        cmd += ["-isystem", d]
    cmd += [MARSHAL_SOURCE, "-o", out, "-L", os.path.join(torch_dir, "lib")]
    return cmd + ["-l" + lib for lib in ("torch_python", "torch", "torch_cpu", "torch_hip", "c10", "c10_hip")]


def build_lib(verbose: bool = False) -> str:
    """Compiles every source to an object (in parallel), links libhq.so and builds _marshal.so."""
    from concurrent.futures import ThreadPoolExecutor

    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    objdir = os.path.join(PKG, "_build")
    os.makedirs(objdir, exist_ok=True)
    inc = ["-I", os.path.join(ROOT, "include"), "-I", CSRC]
    objs = [os.path.join(objdir, os.path.basename(s) + ".%d.o" % os.getpid()) for s in sources()]
    jobs = [[hipcc] + HIPCC_FLAGS + inc + ["-c", src, "-o", obj] for src, obj in zip(sources(), objs)]
    marshal_tmp = MARSHAL + ".tmp%d" % os.getpid()
    jobs.insert(0, marshal_command(marshal_tmp))
    with ThreadPoolExecutor(max_workers=min(8, len(jobs))) as pool:
        list(pool.map(lambda c: _run(c, verbose), jobs))
    tmp = LIB + ".tmp%d" % os.getpid()
    _run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp] + objs, verbose)
    for o in objs:
        os.remove(o)
    os.replace(tmp, LIB)
    os.replace(marshal_tmp, MARSHAL)
    return LIB


if __name__ == "__main__":
    print(build_lib(verbose=True))

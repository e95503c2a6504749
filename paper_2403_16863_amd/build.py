"""Compile the HIP sources of this package for gfx950 into libattn.so, and the native call path of the
binding into _native.so (both in-tree)."""
from __future__ import annotations

import os
import subprocess
import sysconfig
import tempfile
from concurrent.futures import ThreadPoolExecutor

_HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(_HERE, "csrc")
OUT = os.path.join(_HERE, "libattn.so")
NATIVE = os.path.join(_HERE, "_native.so")

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # keep the compiler from forming packed-fp32 VALU instructions
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # kernel arguments arrive in scalar registers (csrc/attn_kernel.h)
    "-mllvm", "-amdgpu-kernarg-preload-count=16",
]
ATTN_PARTS = 9          # parts of the attention variant table (csrc/attn_variants.h)

# (object, source, extra flags)
UNITS = [("attn_fwd.o", "attn_fwd.hip", []), ("gemm_lrelu.o", "gemm_lrelu.hip", [])] + \
        [(f"attn_kernels_{p}.o", "attn_kernels.hip", [f"-DATTN_PART={p}"]) for p in range(ATTN_PARTS)]


def _run(cmd, verbose):
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, cwd=CSRC, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"{cmd[0]} failed:\n{res.stdout}\n{res.stderr}")


def build_native(verbose: bool = False) -> str:
    import torch
    root = os.path.dirname(torch.__file__)
    inc = [os.path.join(root, "include"), os.path.join(root, "include", "torch", "csrc", "api", "include"),
           os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "include"), sysconfig.get_paths()["include"]]
    _run(["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1", *(f"-I{p}" for p in inc),
          f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", "native.cpp", "-o", NATIVE,
          f"-L{os.path.join(root, 'lib')}", "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_python"], verbose)
    return NATIVE


def build_library(verbose: bool = False) -> str:
    jobs = min(len(UNITS), os.cpu_count() or 1, 8)
    with tempfile.TemporaryDirectory(prefix="attn_build_") as tmp:
        with ThreadPoolExecutor(jobs) as pool:
            native = pool.submit(build_native, verbose)
            list(pool.map(lambda u: _run(["hipcc", *HIPCC_FLAGS, *u[2], "-c", "-o", os.path.join(tmp, u[0]), u[1]], verbose),
                          sorted(UNITS, key=lambda u: not u[2])))
            native.result()
        _run(["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", OUT, *(os.path.join(tmp, u[0]) for u in UNITS)], verbose)
    return OUT


if __name__ == "__main__":
    print(build_library(verbose=True))

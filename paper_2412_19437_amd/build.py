"""Build libds3.so (HIP, gfx950 only) in-tree with hipcc.

`python -m paper_2412_19437_amd.build` or `build_library()`.  The shared
library lands in paper_2412_19437_amd/lib/ and is what the Python binding,
the tests and the benchmark load.
"""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIBDIR = os.path.join(HERE, "lib")
LIB = os.path.join(LIBDIR, "libds3.so")
SOURCES = ["ds3_api.hip", "ds3_quant.hip", "ds3_gemm.hip", "ds3_gemm_skinny.hip", "ds3_gemm_shortk.hip", "ds3_probe.hip"]

# -ffp-contract=off: the quantizers' FP32 operation sequence is a bit-exact
#   contract; FMAs in the GEMM are written explicitly.
# packed-fp32-ops off: no v_pk_*_f32 instructions are generated.
# amdgpu-mfma-vgpr-form: MFMA results go to architectural VGPRs, where the
#   per-K-block rescale reads them, instead of AccVGPRs plus copies.
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-ffp-contract=off",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-mllvm", "-amdgpu-mfma-vgpr-form",
    "-Wall", "-Wno-unused-command-line-argument",
]


def _hipcc() -> str:
    exe = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(exe):
        raise RuntimeError("hipcc not found; libds3 needs ROCm to build")
    return exe


def _compile(src: str, objdir: str) -> str:
    obj = os.path.join(objdir, src.replace(".hip", ".o"))
    cmd = [_hipcc(), *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    err = "\n".join(l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{err}")
    if err.strip():
        print(err, file=sys.stderr)
    return obj


def _compile_binding() -> str:
    """ds3_native.so: the Python functions' native marshalling, a host-only extension module against torch's C++ API."""
    import torch
    from torch.utils import cpp_extension
    inc = [*cpp_extension.include_paths("cuda"), sysconfig.get_paths()["include"]]
    out = os.path.join(LIBDIR, "ds3_native.so")
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden", "-D__HIP_PLATFORM_AMD__=1",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", *(f"-isystem{d}" for d in inc),
           os.path.join(CSRC, "ds3_binding.cpp"), "-o", out, f"-L{LIBDIR}", "-lds3",
           f"-L{os.path.join(os.path.dirname(torch.__file__), 'lib')}", "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_python",
           "-Wl,-rpath,$ORIGIN"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("g++ failed on ds3_binding.cpp:\n" + r.stderr)
    return out


def build_library(verbose: bool = True) -> str:
    objdir = os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)
    os.makedirs(LIBDIR, exist_ok=True)
    with ThreadPoolExecutor(max_workers=len(SOURCES)) as ex:
        objs = list(ex.map(lambda s: _compile(s, objdir), SOURCES))
    cmd = [_hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", LIB]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n" + r.stderr)
    _compile_binding()
    if verbose:
        print("built", LIB)
    return LIB


if __name__ == "__main__":
    build_library()

"""Build the C-ABI library (libusp.so) for gfx950 with hipcc, and the binding's calls with g++, in-tree.

    python -m paper_2602_10940_amd.build          # rebuild
"""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
OBJ_DIR = os.path.join(PKG, "_build")
LIB = os.path.join(PKG, "libusp.so")

SOURCES = ["usp_api.hip", "fp8_kernels.hip", "merge_kernel.hip", "attn_generic.hip", "attn_generic_f32.hip", "attn_mfma.hip"]
# libusp_diag.so: the MFMA-rate probe of the benchmark and a test hook, outside the library's ABI
DIAG_LIB = os.path.join(PKG, "libusp_diag.so")
DIAG_SOURCES = [os.path.join("diag", "usp_diag.hip")]

# -packed-fp32-ops off: keep the compiler from forming packed fp32 VALU ops.
# IEEE fp32 division / denormals are required by the FP8 scale arithmetic (no fast-math).
# _usp_calls.so: the binding's calls on torch tensors, a CPython extension (host code) linked against libusp.so
CALLS_LIB = os.path.join(PKG, "_usp_calls.so")
CALLS_SOURCE = "py_calls.cpp"
HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-fhip-fp32-correctly-rounded-divide-sqrt", "-fno-gpu-flush-denormals-to-zero",
    "-fno-fast-math", "-ffp-contract=off",
    # the first 16 words of a kernel's arguments arrive in scalar registers: the scalar cache is cold at every launch, and a
    # kernel of a few microseconds waits ~700 cycles for its first argument (payload of 4608 rows 16.8 -> 16.3 us, merge 4.40 -> 4.25)
    "-mllvm", "-amdgpu-kernarg-preload-count=16",
    "-Wno-unused-command-line-argument", "-Wno-unknown-warning-option",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
]


def hipcc() -> str:
    for c in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if c and (os.path.sep not in c or os.path.exists(c)):
            return c
    raise RuntimeError("hipcc not found")


def hip_include() -> str:
    """The include directory of the ROCm that hipcc() belongs to (a name without a path is looked up as the shell does),
    of torch's, or the usual one: the first that holds HIP's headers."""
    from torch.utils.cpp_extension import ROCM_HOME
    c = shutil.which(hipcc())
    for root in (c and os.path.dirname(os.path.dirname(os.path.realpath(c))), ROCM_HOME, "/opt/rocm"):
        if root and os.path.exists(os.path.join(root, "include", "hip", "hip_runtime_api.h")):
            return os.path.join(root, "include")
    raise RuntimeError("no HIP headers beside hipcc (%s), in ROCM_HOME or under /opt/rocm" % (c or "not on PATH"))


def _compile(src: str, extra) -> str:
    obj = os.path.join(OBJ_DIR, os.path.splitext(os.path.basename(src))[0] + ".o")
    cmd = [hipcc(), *HIPCC_FLAGS, *extra, "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("hipcc failed for %s:\n%s\n%s" % (src, " ".join(cmd), r.stderr[-8000:]))
    return obj


def _compile_calls() -> str:
    import torch
    from torch.utils.cpp_extension import include_paths
    obj = os.path.join(OBJ_DIR, "py_calls.o")
    incs = [sysconfig.get_path("include"), *include_paths(), hip_include(), os.path.join(ROOT, "include")]
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-fvisibility=hidden", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM", "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch._C._GLIBCXX_USE_CXX11_ABI,
           *[x for i in incs for x in ("-isystem", i)], "-c", os.path.join(CSRC, CALLS_SOURCE), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("g++ failed for %s:\n%s\n%s" % (CALLS_SOURCE, " ".join(cmd), r.stderr[-8000:]))
    return obj


def _link_calls(obj: str) -> None:
    import torch
    lib_dir = os.path.join(os.path.dirname(torch.__file__), "lib")
    cmd = ["g++", "-shared", "-fPIC", "-o", CALLS_LIB, obj, "-L", PKG, "-lusp", "-Wl,-rpath,$ORIGIN",
           "-L", lib_dir, "-ltorch_python", "-ltorch", "-ltorch_cpu", "-lc10_hip", "-lc10"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n%s" % r.stderr[-8000:])


def build(verbose: bool = False, extra_flags=()) -> str:
    os.makedirs(OBJ_DIR, exist_ok=True)
    srcs = SOURCES + DIAG_SOURCES
    with ThreadPoolExecutor(max_workers=min(8, len(srcs) + 1)) as ex:
        calls = ex.submit(_compile_calls)
        objs = list(ex.map(lambda s: _compile(s, list(extra_flags)), srcs))
        calls_obj = calls.result()
    n = len(SOURCES)
    for lib, lib_objs, extra in ((LIB, objs[:n], []),
                                 (DIAG_LIB, objs[n:], ["-L", PKG, "-lusp", "-Wl,-rpath,$ORIGIN"])):
        cmd = [hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", "-o", lib, *lib_objs, *extra]
        r = subprocess.run(cmd, capture_output=True, text=True)
        if r.returncode != 0:
            raise RuntimeError("link failed:\n%s" % r.stderr[-8000:])
        if verbose:
            print("built", lib)
    _link_calls(calls_obj)
    if verbose:
        print("built", CALLS_LIB)
    return LIB


if __name__ == "__main__":
    build(verbose=True, extra_flags=sys.argv[1:])

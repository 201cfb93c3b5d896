"""Build libqwam.so (HIP kernels for gfx950 + the C ABI) in-tree with hipcc, and
the CPython module of its per-token calls (_qwam_call) with the host compiler.
The library needs hipcc only.  The module also needs g++ and PyTorch's headers;
when it does not build, the library is linked all the same and the error follows.

Usage: python -m paper_2609_33269_amd.build [-v]
"""

from __future__ import annotations

import concurrent.futures as cf
import os
import shutil
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
BUILD_DIR = os.path.join(ROOT, "_build")
LIB = os.path.join(HERE, "libqwam.so")
CALL_MODULE = os.path.join(HERE, "_qwam_call.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
ARCH = "gfx950"

SOURCES = ["qwam_api.cpp", "qwam_quant.hip", "qwam_rotate.hip", "qwam_aog.hip", "qwam_gemm.hip", "qwam_gemm_mid.hip", "qwam_gemm_small.hip",
           "qwam_layer_small.hip", "qwam_probe.hip", "qwam_eig.hip"]

# Packed-FP32 VALU instructions are disabled on purpose (some of their forms
# have produced silently wrong results on this hardware).  No fast-math: the
# quantizer relies on correctly rounded division and IEEE float32 semantics.
COMMON_FLAGS = [
    "-O3", "-std=c++17", "-fPIC", f"--offload-arch={ARCH}",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
    f"-I{os.path.join(ROOT, 'include')}",
]


def _compile(src: str, verbose: bool) -> str:
    obj = os.path.join(BUILD_DIR, os.path.splitext(src)[0] + ".o")
    cmd = [HIPCC, *COMMON_FLAGS]
    if src.endswith(".cpp"):
        cmd += ["-x", "hip"]
    cmd += ["-c", os.path.join(CSRC, src), "-o", obj]
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    msgs = "\n".join(l for l in (res.stdout + res.stderr).splitlines()
                     if "is not a recognized feature for this target" not in l)
    if res.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{msgs}")
    if verbose and msgs.strip():
        print(msgs, flush=True)
    return obj


def _rocm_root() -> str:
    """The ROCm installation of HIPCC, which may be a path, a link or a name on PATH."""
    path = shutil.which(HIPCC)
    if path is None:
        raise RuntimeError(f"{HIPCC}: no such program")
    for p in (path, os.path.realpath(path)):
        root = os.path.dirname(os.path.dirname(os.path.abspath(p)))
        if os.path.exists(os.path.join(root, "include", "hip", "hip_runtime.h")):
            return root
    raise RuntimeError(f"no HIP headers beside {path}")


def _build_call_module(verbose: bool) -> None:
    import torch
    tdir = os.path.dirname(torch.__file__)
    rocm = _rocm_root()
    tmp = CALL_MODULE + ".tmp"
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", "-DUSE_ROCM", "-D__HIP_PLATFORM_AMD__",
           "-isystem", f"{tdir}/include", "-isystem", f"{tdir}/include/torch/csrc/api/include",
           "-isystem", f"{rocm}/include", "-isystem", sysconfig.get_paths()["include"],
           os.path.join(CSRC, "qwam_binding.cpp"), "-o", tmp,
           f"-L{tdir}/lib", "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip", f"-Wl,-rpath,{tdir}/lib"]
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"g++ failed on qwam_binding.cpp:\n{res.stdout}\n{res.stderr}")
    os.replace(tmp, CALL_MODULE)


def build(verbose: bool = False) -> str:
    """Compile every source, link libqwam.so and the call module; returns the
    library path."""
    os.makedirs(BUILD_DIR, exist_ok=True)
    with cf.ThreadPoolExecutor(max_workers=len(SOURCES) + 1) as ex:
        call = ex.submit(_build_call_module, verbose)
        objs = list(ex.map(lambda s: _compile(s, verbose), SOURCES))
    tmp = LIB + ".tmp"
    cmd = [HIPCC, f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", tmp, *objs]
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"link failed:\n{res.stdout}\n{res.stderr}")
    os.replace(tmp, LIB)
    call.result()       # the module's error, if any
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))

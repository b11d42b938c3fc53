"""Build libfalqon.so (HIP, gfx950 only) in-tree with hipcc, and _calls.so, the Python extension through which the
calls of a training step reach it, with the host compiler against the installed torch.

    python -m paper_2510_24061_amd.build

Objects go to paper_2510_24061_amd/_build/ (git-ignored); the libraries land next to this
file so that they travel with the source tree.
"""
import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
BUILD = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libfalqon.so")
SOURCES = ["falqon_api.hip", "quantize.hip", "gemm.hip", "gemm_mid.hip", "gemm_thin.hip", "partials.hip", "db.hip", "proxy.hip", "optimizer.hip", "init.hip",
           "db_wide.hip"]
CALLS = os.path.join(HERE, "_calls.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",   # never emit packed-fp32 VALU ops
    "-Wall", "-Wno-unused-command-line-argument",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
]


def _compile(src: str) -> str:
    obj = os.path.join(BUILD, os.path.splitext(src)[0] + ".o")
    cmd = [HIPCC, *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    noise = "is not a recognized feature for this target"
    err = "\n".join(l for l in r.stderr.splitlines() if noise not in l)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{err}")
    if err.strip():
        sys.stderr.write(err + "\n")
    return obj


def _build_calls() -> None:
    import torch
    from torch.utils import cpp_extension
    includes = [*cpp_extension.include_paths(), sysconfig.get_paths()["include"]]
    tmp = CALLS + ".tmp"
    subprocess.run([os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall",
                    f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
                    "-I", os.path.join(ROOT, "include"), *(a for d in includes for a in ("-isystem", d)),
                    os.path.join(CSRC, "python_calls.cpp"), "-o", tmp,
                    *(a for d in cpp_extension.library_paths() for a in ("-L", d)), "-ltorch_python", "-ltorch_cpu", "-lc10",
                    "-L", HERE, "-l:libfalqon.so", "-Wl,-rpath,$ORIGIN"], check=True)
    os.replace(tmp, CALLS)


def build() -> str:
    os.makedirs(BUILD, exist_ok=True)
    with ThreadPoolExecutor(max_workers=min(8, len(SOURCES))) as ex:
        objs = list(ex.map(_compile, SOURCES))
    tmp = LIB + ".tmp"
    subprocess.run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp, *objs], check=True)
    os.replace(tmp, LIB)
    _build_calls()
    return LIB


if __name__ == "__main__":
    print(build())

"""Build libjz.so (HIP kernels + C ABI) for gfx950 and the binding's native part in-tree: python -m paper_1807_11205_amd.build

Every csrc/*.hip is compiled to an object of its own, in parallel, then linked; objects go to a scratch directory
outside the source tree."""
import glob
import os
import subprocess
import sys
import sysconfig
import tempfile
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
OUT = os.path.join(PKG, "libjz.so")
HOST_OUT = os.path.join(PKG, "_jz_host.so")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fno-gpu-rdc",
    # keep the compiler from forming packed-fp32 VALU instructions
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function", "-Wno-cuda-compat",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
]


def build_host(verbose: bool = False) -> str:
    """csrc/jz_host.cpp, the CPython module the binding imports."""
    import torch
    t = os.path.dirname(os.path.abspath(torch.__file__))
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-shared", "-fPIC", "-Wall", "-I", os.path.join(ROOT, "include"),
           "-I", sysconfig.get_paths()["include"], "-isystem", os.path.join(t, "include"),
           "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI), "-o", HOST_OUT, os.path.join(CSRC, "jz_host.cpp"),
           "-L", os.path.join(t, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10"]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    return HOST_OUT


def build(verbose: bool = False, extra=()) -> str:
    srcs = sorted(glob.glob(os.path.join(CSRC, "*.hip")))
    jobs = max(1, min(len(srcs), int(os.environ.get("MAX_JOBS", "0")) or os.cpu_count() or 1, 16))
    with tempfile.TemporaryDirectory(prefix="jzbuild_") as tmp:
        def compile_one(src):
            obj = os.path.join(tmp, os.path.basename(src)[:-4] + ".o")
            cmd = [HIPCC, *FLAGS, *extra, "-c", "-o", obj, src]
            if verbose:
                print(" ".join(cmd), flush=True)
            subprocess.run(cmd, check=True)
            return obj

        with ThreadPoolExecutor(jobs + 1) as pool:
            host = pool.submit(build_host, verbose)
            objs = list(pool.map(compile_one, srcs))
            host.result()
        link = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-fno-gpu-rdc", "-o", OUT, *objs]
        if verbose:
            print(" ".join(link), flush=True)
        subprocess.run(link, check=True)
    return OUT


if __name__ == "__main__":
    print(build(verbose=True, extra=sys.argv[1:]))

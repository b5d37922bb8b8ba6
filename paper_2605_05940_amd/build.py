"""Compile the HIP sources under ``csrc/`` into ``libnpd.so`` for gfx950 (cross-compiles without a GPU), and the binding's
native argument marshalling (``npd_host.cpp``, host code against the installed torch) into ``npd_host.so``."""
import concurrent.futures
import glob
import os
import shutil
import subprocess
import sys
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libnpd.so")
HOST = os.path.join(HERE, "npd_host.so")

HIPCC_FLAGS = [
    "-O3", "-std=c++17", "-fPIC", "--offload-arch=gfx950",
    # packed fp32 VALU forms are kept out of the generated code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # no implicit fusing of a*b+c: every fused multiply-add in the kernels is written out, so that two
    # streams fed the same data round the same way wherever the expression is inlined
    "-ffp-contract=off",
    "-Wall", "-Wno-unused-command-line-argument",
]


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def build_host(verbose: bool = False) -> str:
    import sysconfig
    import torch
    root = os.path.dirname(torch.__file__)
    lib = os.path.join(root, "lib")
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden", "-Wall",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch.compiled_with_cxx11_abi())}",
           "-isystem", os.path.join(root, "include"), "-isystem", sysconfig.get_paths()["include"],
           os.path.join(CSRC, "npd_host.cpp"), "-o", HOST, "-L" + lib, "-lc10", "-ltorch_cpu", "-ltorch", "-ltorch_python",
           "-Wl,-rpath," + lib]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    return HOST


def build(verbose: bool = False, extra=(), out: str = LIB, jobs: int = 6) -> str:
    """Every source becomes an object of its own (in parallel), then one shared library."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    tmp = tempfile.mkdtemp(prefix="npd_build_")
    try:
        def compile_one(src):
            obj = os.path.join(tmp, os.path.basename(src)[:-4] + ".o")
            cmd = [hipcc, *HIPCC_FLAGS, *extra, "-c", src, "-o", obj]
            if verbose:
                print(" ".join(cmd), flush=True)
            subprocess.check_call(cmd)
            return obj
        with concurrent.futures.ThreadPoolExecutor(max_workers=jobs) as pool:
            host = pool.submit(build_host, verbose) if out == LIB else None
            objs = list(pool.map(compile_one, sources()))
            if host:
                host.result()
        cmd = [hipcc, "-shared", "-fPIC", "--offload-arch=gfx950", "-o", out, *objs]
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.check_call(cmd)
    finally:
        shutil.rmtree(tmp, ignore_errors=True)
    return out


if __name__ == "__main__":
    print(build(verbose=True, extra=sys.argv[1:]))

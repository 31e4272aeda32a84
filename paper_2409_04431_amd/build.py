"""Compile the HIP library for gfx950 with hipcc (cross-compiles without a GPU) and the native half of
the Python binding with g++ against it."""
import os
import subprocess
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libsattn.so")
NATIVE = os.path.join(HERE, "_native.so")
# one translation unit per head dimension and direction, so the kernels compile in parallel
SOURCES = ["sattn_api.hip", "sattn_fwd_d64.hip", "sattn_fwd_d128.hip", "sattn_bwd_d64.hip", "sattn_bwd_d128.hip"]

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    # packed fp32 VALU ops are kept off for every kernel in this library
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
]


def _run(cmd):
    res = subprocess.run(cmd, capture_output=True, text=True)
    err = "\n".join(l for l in res.stderr.splitlines() if "is not a recognized feature" not in l)
    if res.returncode != 0:
        raise RuntimeError("compilation failed:\n" + " ".join(cmd) + "\n" + err)
    return err


def _build_native():
    import torch

    root = os.path.dirname(torch.__file__)
    return _run([os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall",
                 f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
                 "-isystem", os.path.join(root, "include"),
                 "-isystem", os.path.join(root, "include", "torch", "csrc", "api", "include"),
                 "-isystem", sysconfig.get_paths()["include"],
                 "-o", NATIVE, os.path.join(CSRC, "binding_native.cpp"),
                 "-L" + os.path.join(root, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10",
                 "-L" + HERE, "-lsattn", "-Wl,-rpath,$ORIGIN"])


def build_library(verbose=False, jobs=None):
    """(Re)build libsattn.so and _native.so in-tree.  Always compiles every source."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    os.makedirs(OBJ, exist_ok=True)
    compile_flags = [f for f in HIPCC_FLAGS if f != "-shared"]
    objs = [os.path.join(OBJ, s + ".o") for s in SOURCES]
    cmds = [[hipcc] + compile_flags + ["-c", "-o", o, os.path.join(CSRC, s)] for s, o in zip(SOURCES, objs)]
    jobs = jobs or min(len(cmds), os.cpu_count() or 1, 16)
    with ThreadPoolExecutor(max_workers=jobs) as pool:
        msgs = list(pool.map(_run, cmds))
    msgs.append(_run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB] + objs))
    msgs.append(_build_native())
    if verbose and any(m.strip() for m in msgs):
        print("\n".join(m for m in msgs if m.strip()))
    return LIB


if __name__ == "__main__":
    print(build_library(verbose=True))

"""Compile the HIP libraries for gfx950: csrc/medha.hip into libmedha.so (the product)
and csrc/yardstick.hip into libmedha_yardstick.so (the benchmark's yardsticks), and the
binding's host code, csrc/marshal.cpp, into the extension module _marshal.

The libraries need hipcc alone.  The module needs g++, the headers of this interpreter (Python 3.10
or later) and of torch, and works with the interpreter and the torch that it is built with: its
file name carries the one's tag and its torch_version names the other.

Run as ``python -m paper_2409_17264_amd.build``; also called by
``__graft_entry__.build()``.  hipcc cross-compiles without a GPU.
"""
import glob
import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(os.path.dirname(HERE), "include")
LIB = os.path.join(HERE, "libmedha.so")
# source file -> shared library
TARGETS = {"medha.hip": LIB, "yardstick.hip": os.path.join(HERE, "libmedha_yardstick.so")}

MARSHAL = os.path.join(HERE, "_marshal" + sysconfig.get_config_var("EXT_SUFFIX"))

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function", "-Wno-inline-asm", "-fno-gpu-rdc",
]


def _run(cmd, what: str, verbose: bool) -> None:
    if verbose:
        print(" ".join(cmd))
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        sys.stderr.write(res.stdout + res.stderr)
        raise RuntimeError(f"the compiler failed on {what}")
    if verbose and res.stderr:
        lines = [l for l in res.stderr.splitlines() if "packed-fp32-ops" not in l]
        sys.stderr.write("\n".join(lines) + "\n")


def _marshal_command():
    import torch

    root = os.path.dirname(torch.__file__)
    include, lib = os.path.join(root, "include"), os.path.join(root, "lib")
    return [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall",
            f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
            f'-DMEDHA_TORCH_VERSION="{torch.__version__}"',
            "-I", INCLUDE, "-I", CSRC, "-isystem", include,
            "-isystem", os.path.join(include, "torch", "csrc", "api", "include"),
            "-isystem", sysconfig.get_paths()["include"], os.path.join(CSRC, "marshal.cpp"),
            "-o", MARSHAL, "-L", lib, "-lc10", "-ltorch_cpu", "-ltorch_python"]


def build(verbose: bool = False) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    found = sorted(os.path.basename(p) for p in glob.glob(os.path.join(CSRC, "*.hip")))
    assert found == sorted(TARGETS), f"every .hip source needs a target: {found}"
    for src, lib in TARGETS.items():
        _run([hipcc] + HIPCC_FLAGS + ["-I", INCLUDE, "-I", CSRC, os.path.join(CSRC, src), "-o", lib],
             src, verbose)
    _run(_marshal_command(), "marshal.cpp", verbose)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))

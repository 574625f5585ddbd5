"""Builds libshampoo.so (HIP, gfx950 only) and _marshal.so (host code) next to this file.

    python -m paper_2309_06497_amd.build
"""
import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
LIB = os.path.join(HERE, "libshampoo.so")
MARSHAL = os.path.join(HERE, "_marshal.so")
SOURCES = [os.path.join(HERE, "csrc", "shampoo.hip")]
FLAGS = [
    "-O3", "-std=c++17", "-fPIC", "-shared", "--offload-arch=gfx950",
    # packed fp32 instructions are kept out of the generated code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
]


def marshal_command():
    """g++ line of the extension that checks a step's tensors (csrc/marshal.cpp)."""
    import torch
    root = os.path.dirname(torch.__file__)
    inc = [os.path.join(root, "include"), os.path.join(root, "include", "torch", "csrc", "api", "include"),
           os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "include"), sysconfig.get_paths()["include"]]
    return (["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-w", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
             "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI)]
            + ["-isystem" + i for i in inc] + [os.path.join(HERE, "csrc", "marshal.cpp"), "-o", MARSHAL,
               "-L" + os.path.join(root, "lib"), "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_python"])


def build(verbose=True):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    cmds = [[hipcc] + FLAGS + SOURCES + ["-o", LIB], marshal_command()]
    for cmd in cmds:
        if verbose:
            print(" ".join(cmd), flush=True)
    running = [subprocess.Popen(cmd) for cmd in cmds]     # side by side
    failed = [cmd for cmd, p in zip(cmds, running) if p.wait() != 0]
    if failed:
        raise subprocess.CalledProcessError(1, failed[0])
    return LIB


if __name__ == "__main__":
    build()
    sys.exit(0)

"""The reciprocal and the reciprocal square root of csrc/eigh_jacobi.h, compiled for the CPU with estimates that are wrong by 2^-24 either
way, as those of the hardware are."""
import os
import re
import subprocess

import numpy as np
import pytest

HEADER = os.path.join(os.path.dirname(os.path.abspath(__file__)), "..", "paper_2309_06497_amd", "csrc", "eigh_jacobi.h")


@pytest.fixture(scope="module")
def functions(tmp_path_factory):
    import ctypes
    text = open(HEADER).read()
    body = "".join(re.search(r"__device__ __forceinline__ double %s\(double x\) \{.*?\n\}\n" % name, text, re.S).group(0) for name in ("rsqrt_newton", "rcp_newton"))
    folder = tmp_path_factory.mktemp("steps")
    src, lib = str(folder / "steps.cpp"), str(folder / "steps.so")
    with open(src, "w") as f:
        f.write("#include <cmath>\n#define __device__\n#define __forceinline__ inline\nstatic double off;\n"
                "static double __builtin_amdgcn_rsq(double x) { return (1.0 + off) / std::sqrt(x); }\n"
                "static double __builtin_amdgcn_rcp(double x) { return (1.0 + off) / x; }\n" + body +
                'extern "C" double rsqrt_of(double x, double o) { off = o; return rsqrt_newton(x); }\n'
                'extern "C" double rcp_of(double x, double o) { off = o; return rcp_newton(x); }\n')
    subprocess.run(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", "-ffp-contract=off", src, "-o", lib], check=True)
    so = ctypes.CDLL(lib)
    for f in (so.rsqrt_of, so.rcp_of):
        f.restype, f.argtypes = ctypes.c_double, [ctypes.c_double, ctypes.c_double]
    return so


@pytest.mark.parametrize("off", [2.0 ** -24, -2.0 ** -24])
def test_two_steps_reach_float64(functions, off):
    r = np.random.default_rng(0)
    # a step leaves 1.5 times the square of the error, and a few roundings of 2^-53
    for x in np.exp2(r.uniform(-1021, 1023, 5000)):
        assert abs(np.longdouble(functions.rsqrt_of(x, off)) * np.sqrt(np.longdouble(x)) - 1) <= 2.0 ** -50, x
    for x in np.exp2(r.uniform(-1021, 1021, 5000)):
        assert abs(np.longdouble(functions.rcp_of(x, off)) * np.longdouble(x) - 1) <= 2.0 ** -50, x


@pytest.mark.parametrize("off", [2.0 ** -24, -2.0 ** -24])
def test_roots_of_subnormal_numbers(functions, off):
    """Half of x rounds to a multiple of 2^-1074, which is all that the result loses."""
    for e in range(1024, 1073):
        for m in (1.0, 1.3, 1.9):
            x = m * 2.0 ** -e
            err = abs(np.longdouble(functions.rsqrt_of(x, off)) * np.sqrt(np.longdouble(x)) - 1)
            assert err <= 2.0 ** -50 + 2.0 ** -1074 / x, (e, m, err)

"""The rule that cuts the Gram matrices of tensor blocks into ranges (csrc/gram_split.h), compiled for the host: over
the shapes that a block can have, the ranges cover k, none is empty, and their matrices fit the scratch of the block."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2309_06497_amd", "csrc")
SHIM = r"""
#include "gram_split.h"
#include <cstdio>
using shampoo::gram_split;
// number of (K, room, workgroups) whose split is not sound, among them the first one
extern "C" long long faults(int32_t lo, int32_t hi, int64_t workgroups, int64_t *first) {
  long long bad = 0;
  for (int64_t K = lo; K < hi; ++K)
    for (int64_t room = 1; room <= 80; ++room) {
      const shampoo::GramSplit s = gram_split(K, room, workgroups, 16);
      const bool ok = s.ranges == 1 ? s.range >= K
                                    : s.ranges <= room && s.range % 16 == 0 && s.range >= 64 &&
                                          (int64_t)s.ranges * s.range >= K && (int64_t)(s.ranges - 1) * s.range < K;
      if (!ok && bad++ == 0) { first[0] = K; first[1] = room; first[2] = s.ranges; first[3] = s.range; }
    }
  return bad;
}
extern "C" int ranges(int64_t K, int64_t room, int64_t workgroups) { return gram_split(K, room, workgroups, 16).ranges; }
"""


@pytest.fixture(scope="module")
def shim(tmp_path_factory):
    d = tmp_path_factory.mktemp("gram_split")
    src, lib = d / "shim.cpp", d / "shim.so"
    src.write_text(SHIM)
    subprocess.run(["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-I" + CSRC, str(src), "-o", str(lib)], check=True)
    L = ctypes.CDLL(str(lib))
    L.faults.restype = ctypes.c_longlong
    L.faults.argtypes = [ctypes.c_int32, ctypes.c_int32, ctypes.c_int64, ctypes.POINTER(ctypes.c_int64)]
    L.ranges.argtypes = [ctypes.c_int64] * 3
    return L


@pytest.mark.parametrize("workgroups", [1, 3, 16, 100, 117, 341, 1000, 5000])
def test_ranges_cover_k_and_fit_the_scratch(shim, workgroups):
    first = (ctypes.c_int64 * 4)()
    bad = shim.faults(1, 20000, workgroups, first)
    assert bad == 0, f"{bad} bad splits; K, room, ranges, range of the first: {list(first)}"


def test_a_72_by_64_by_9_block(shim):
    """k = 72 * 9 of the middle dimension, room for 10 matrices of 64 x 64: a range of floor(648 / 10) = 64 values
    would make eleven."""
    assert shim.ranges(648, 72 * 64 * 9 // (64 * 64), 1) <= 10

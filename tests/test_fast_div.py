"""The division by multiplication that the kernels' index arithmetic uses (FastDiv), compiled for the CPU from the header the kernels include
and compared with integer division at the edges of its range (0 <= n < 2^31, 1 <= d < 2^31): multiples of d and their
neighbours, powers of two, the largest n."""
import ctypes
import os
import random
import shutil
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2409_12490_amd", "csrc")
PROGRAM = """
#define __host__
#define __device__
#define __forceinline__ inline
#include "fast_div.h"
extern "C" void divide(uint32_t d, const uint32_t* n, uint32_t* out, int count) {
    const cp::FastDiv f(d);
    for (int i = 0; i < count; ++i) out[i] = f.div(n[i]);
}
"""


@pytest.fixture(scope="module")
def divide(tmp_path_factory):
    compiler = shutil.which("g++") or shutil.which("clang++") or shutil.which("c++")
    if compiler is None:
        pytest.skip("no C++ compiler")
    where = tmp_path_factory.mktemp("fast_div")
    (where / "f.cpp").write_text(PROGRAM)
    subprocess.run([compiler, "-O1", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, str(where / "f.cpp"), "-o", str(where / "f.so")], check=True)
    lib = ctypes.CDLL(str(where / "f.so"))
    u32 = np.ctypeslib.ndpointer(np.uint32)
    lib.divide.argtypes = [ctypes.c_uint32, u32, u32, ctypes.c_int]
    lib.divide.restype = None
    return lib.divide


def test_exact_over_the_range(divide):
    g = random.Random(1)
    top = (1 << 31) - 1
    divisors = [1, 2, 3, 5, 7, 255, 256, 257, 65535, 65537, top, top - 1, 1 << 30, (1 << 30) + 1]
    divisors += [g.randrange(1, 1 << g.randrange(1, 31)) for _ in range(400)]
    for d in divisors:
        ns = {0, 1, d - 1, d, min(top, d + 1), top, top // d * d, max(0, top // d * d - 1)}
        for _ in range(50):
            x = d * g.randrange(0, top // d + 1)
            ns |= {x, max(0, x - 1), min(top, x + 1), g.randrange(0, top + 1)}
        n = np.array(sorted(ns), dtype=np.uint32)
        out = np.empty_like(n)
        divide(d, n, out, len(n))
        np.testing.assert_array_equal(out, n // np.uint32(d), err_msg=str(d))

"""The kernels' division by sizes known at launch (csrc/rbgp_fastdiv.h) against Python's, compiled for the host."""
import ctypes
import os
import random
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2006_13486_amd", "csrc")
SOURCE = """
#define __host__
#define __device__
#define __forceinline__ inline
#include "rbgp_fastdiv.h"
extern "C" int quotient(int n, int64_t d) { return rbgp_fast::quotient(n, rbgp_fast::div_by(d)); }
"""


@pytest.fixture(scope="module")
def quotient(tmp_path_factory):
    d = tmp_path_factory.mktemp("fastdiv")
    src, lib = d / "q.cpp", d / "q.so"
    src.write_text(SOURCE)
    subprocess.check_call(["g++", "-O1", "-shared", "-fPIC", "-I", CSRC, "-o", str(lib), str(src)])
    fn = ctypes.CDLL(str(lib)).quotient
    fn.argtypes, fn.restype = [ctypes.c_int, ctypes.c_int64], ctypes.c_int
    return fn


@pytest.mark.parametrize("divisors", [range(1, 700), [2**k + e for k in range(10, 31) for e in (-1, 0, 1)], None],
                         ids=["small", "around_powers_of_two", "random"])
def test_quotients(quotient, divisors):
    rng = random.Random(5)
    for d in divisors or [rng.randrange(1, 2**31) for _ in range(2000)]:
        last = (2**31 - 1) // d * d   # the largest multiple, and the numbers around it
        for n in {0, 1, d - 1, d, d + 1, 2 * d - 1, 2 * d, last - 1, last, 2**31 - 1, rng.randrange(2**31)}:
            if 0 <= n < 2**31:
                assert quotient(n, d) == n // d, (n, d)

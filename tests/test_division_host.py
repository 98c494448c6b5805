"""The kernels' short division by a number whose reciprocal the host has prepared."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = r"""
#include "lite_attn_kernels.h"
extern "C" long wrong(int b, int from, int to) {  // numerators for which the quotient by b is wrong
  const uint32_t per_b = la::reciprocal(b);
  long n = 0;
  for (long a = from; a < to; ++a) n += la::quotient((int)a, b, per_b) != a / b;
  return n;
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("div")
    (d / "div.cpp").write_text(SRC)
    out = str(d / "libdiv.so")
    subprocess.run(["g++", "-std=c++17", "-O2", "-fPIC", "-shared", "-I" + os.path.join(ROOT, "tests", "hip_stub"),
                    "-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(ROOT, "paper_2511_11062_amd", "csrc"),
                    str(d / "div.cpp"), "-o", out], check=True)
    return ctypes.CDLL(out)


@pytest.mark.parametrize("b", [1, 2, 3, 7, 16, 185, 192, 511, 512, 513, 16383, 65537, 1 << 23, (1 << 30) - 1, 1 << 30])
def test_quotients(lib, b):
    """Rows and segments (up to 2^30 rows in all): from zero, and around multiples of b up to the largest number of rows."""
    lib.wrong.restype = ctypes.c_long
    assert lib.wrong(b, 0, 1 << 20) == 0
    for k in {1, 2, 1000, ((1 << 30) - 1) // b, (1 << 30) // b}:
        at = k * b
        if 0 < at <= 1 << 30:
            assert lib.wrong(b, max(0, at - 3), min(at + 3, 1 << 30)) == 0

"""The learned preconditioner's work array covers every evaluation it is kept for (host arithmetic of
csrc/partials.h, compiled here with the host compiler; no GPU): an array sized for Sa samples serves every
S <= Sa, so its size has to reach what any of them uses."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2407_08901_amd", "csrc")

SRC = r"""
#include "partials.h"
// first n of [n0, n1], step by step, where an S <= Sa <= 32 uses more than the size for Sa; 0: none
extern "C" long short_at(long n0, long n1, long step, int* S_out, int* Sa_out) {
  for (long n = n0; n <= n1; n += step) {
    long most = 0;
    int at = 0;
    for (int Sa = 1; Sa <= 32; ++Sa) {
      const long u = sppc::mpnn_work_used(n, Sa);
      if (u > most) { most = u; at = Sa; }
      if (most > sppc::mpnn_work_doubles(n, Sa)) { *S_out = at; *Sa_out = Sa; return n; }
    }
  }
  return 0;
}
"""


@pytest.fixture(scope="module")
def short_at(tmp_path_factory):
    d = tmp_path_factory.mktemp("sizes")
    (d / "sizes.cpp").write_text(SRC)
    so = str(d / "sizes.so")
    subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, str(d / "sizes.cpp"), "-o", so],
                   check=True)
    f = ctypes.CDLL(so).short_at
    f.restype = ctypes.c_long
    f.argtypes = [ctypes.c_long] * 3 + [ctypes.POINTER(ctypes.c_int)] * 2
    return f


# every row count of the usual sizes, then strides (prime, so that every remainder is met) up to 2^31
@pytest.mark.parametrize("n0,n1,step", [(1, 1000000, 1), (1000001, 40000000, 499), (40000001, (1 << 31) - 1, 99991)])
def test_a_larger_evaluation_s_array_serves_every_smaller_one(short_at, n0, n1, step):
    S, Sa = ctypes.c_int(0), ctypes.c_int(0)
    n = short_at(n0, n1, step, ctypes.byref(S), ctypes.byref(Sa))
    assert n == 0, "n = %d: S = %d needs more than the array sized for %d" % (n, S.value, Sa.value)

"""The row-index divisions of the kernels (csrc/laserkv_index.h), compiled for the host and checked over all limits:
window rows m = g * W + j with G * W <= 1024, block rows m = g * n_q + j with G <= 1024 and n_q <= 16384."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2602_02199_amd", "csrc")
SOURCE = r"""
#include "laserkv_index.h"
static bool bad(int m, int n, uint32_t magic, bool block) {
  int r, q;
  if (block) {
    q = lkv::div_rem(m, n, magic, &r);
  } else {
    q = lkv::div_w(m, magic);
    r = m - q * n;
  }
  return q != m / n || r != m % n;
}
// every m < limit for n == 1 .. n_max
extern "C" long all_rows(int n_max, int limit, int block) {
  long wrong = 0;
  for (int n = 1; n <= n_max; ++n)
    for (int m = 0; m < limit; ++m) wrong += bad(m, n, lkv::div_magic(n), block);
  return wrong;
}
// the first and last rows of heads 0 .. group - 1 for n == 1 .. n_max: the products are monotonic in m, so a quotient
// that is right at both ends of a head is right in between
extern "C" long head_ends(int n_max, int group, int block) {
  long wrong = 0;
  for (int n = 1; n <= n_max; ++n)
    for (int g = 0; g < group; ++g) wrong += bad(g * n, n, lkv::div_magic(n), block) + bad(g * n + n - 1, n, lkv::div_magic(n), block);
  return wrong;
}
"""


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    d = tmp_path_factory.mktemp("index")
    (d / "index.cpp").write_text(SOURCE)
    subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, "-o", str(d / "index.so"), str(d / "index.cpp")], check=True)
    lib = ctypes.CDLL(str(d / "index.so"))
    lib.all_rows.restype = lib.head_ends.restype = ctypes.c_long
    return lib


def test_window_rows(host):
    assert host.all_rows(1024, 1024, 0) == 0


def test_block_rows(host):
    assert host.head_ends(16384, 1024, 1) == 0
    assert host.all_rows(64, 1 << 16, 1) == 0


def test_the_short_division_is_not_enough_for_block_rows(host):
    assert host.head_ends(16384, 16, 0) == 0 and host.head_ends(16384, 32, 0) > 0


def test_the_kernel_of_many_rows_takes_the_long_division():
    src = open(os.path.join(CSRC, "laserkv_attend.hip")).read()
    start = src.index("void attend_rows_kernel")
    body = src[start:src.index("\n__global__", start)]
    assert "div_rem(" in body and "div_w(" not in body

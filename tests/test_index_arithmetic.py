"""The row-index arithmetic of the kernels (csrc/laserkv_index.h), compiled for the host: the divisions over all limits,
window rows m = g * W + j with G * W <= 1024, block rows m = g * n_q + j with G <= 1024 and n_q <= 16384; and the key
ranges of attention launches of many rows against a count by rows."""
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
extern "C" void rows_ranges(int m_rows, int n_q, int cache_len, int s_t, int diag, int pg, int n_splits, int* both, int* share, int* last) {
  const lkv::RowsShape s{m_rows, n_q, lkv::div_magic(n_q), cache_len, s_t, diag};
  *both = lkv::rows_cut(s, pg, n_splits).both;
  *share = lkv::rows_cut(s, pg, n_splits).share;
  *last = lkv::rows_last_cache_range(s, pg, n_splits);
}
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
    lib.rows_ranges.restype = None
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
    index = open(os.path.join(CSRC, "laserkv_index.h")).read()
    body = index[index.index("int rows_tile_end("):]
    assert "div_rem(" in body and "div_w(" not in body


@pytest.mark.parametrize("group,n_q,cache_len,s_t,n_splits", [
    (8, 128, 2400, 4096, 8),   # window rows before a long block: 300 cache rows a split on average, ranges of up to 832 and none
    (4, 128, 63520, 0, 8), (4, 128, 63520, 0, 8), (4, 2048, 910, 2048, 3), (1, 160, 400, 160, 2), (7, 33, 5000, 300, 16), (4, 64, 0, 2048, 4), (2, 250, 333, 1000, 5)])
def test_the_last_cache_range_of_a_cut_row_group(host, group, n_q, cache_len, s_t, n_splits):
    m_rows, diag = group * n_q, s_t - n_q
    n_tiles = (m_rows + 31) // 32
    ends = [max([0] + [min(s_t, diag + m % n_q + 1) for m in range(32 * t, min(32 * t + 32, m_rows))]) for t in range(n_tiles)]
    for pg in range((n_tiles + 7) // 8):
        # units of time of the group's first pair: a cache row or a block key that both of its tiles see, then two keys each
        ea, eb = ends[4 * pg], ends[n_tiles - 1 - 4 * pg]
        units = cache_len + min(ea, eb) + (abs(ea - eb) + 1) // 2
        share = (-(-units // n_splits) + 31) // 32 * 32
        rows = [min(cache_len, (r + 1) * share) - min(cache_len, r * share) for r in range(n_splits)]
        assert rows[-1] == min(rows)
        got = [ctypes.c_int() for _ in range(3)]
        host.rows_ranges(m_rows, n_q, cache_len, s_t, diag, pg, n_splits, *[ctypes.byref(x) for x in got])
        assert [x.value for x in got] == [cache_len + min(ea, eb), share, rows[-1]]


def test_the_instance_with_the_ring_is_chosen_by_the_ranges_that_the_kernel_cuts():
    src = open(os.path.join(CSRC, "laserkv_attend.hip")).read()
    launch = src[src.index("hipError_t launch_attend_t("):]
    assert "rows_last_cache_range(shape, pg, p.n_splits) > 2 * RING_KEYS" in launch[:launch.index("\n}")]
    kernel = src[src.index("void attend_rows_kernel"):]
    assert "rows_cut(shape, pg, n_splits)" in kernel[:kernel.index("\n__global__")]

// Row-index arithmetic of the kernels: plain C++ too, so that it can be checked over all limits without a GPU.
#pragma once

#include <stdint.h>

#if defined(__HIPCC__)
#include <hip/hip_runtime.h>
#define LKV_HD __host__ __device__ __forceinline__
#else
#define LKV_HD inline
#endif

namespace lkv {

// The multiplier of the divisions below, ceil(2^32 / n); n == 1 has none of 32 bits and gets 0.
LKV_HD uint32_t div_magic(int n) { return n > 1 ? (uint32_t)(((uint64_t(1) << 32) + (uint64_t)n - 1) / (uint64_t)n) : 0u; }

LKV_HD int mul_hi(int m, uint32_t magic) { return (int)(((uint64_t)(uint32_t)m * magic) >> 32); }

// m / n, exact while m * n < 2^32: the multiplier exceeds 2^32 / n by less than 1, so the product exceeds m / n by less
// than m / 2^32 <= 1 / n.  Enough for window rows (m < 1024, n <= 1024).
LKV_HD int div_w(int m, uint32_t magic) { return magic ? mul_hi(m, magic) : m; }

// m / n and the remainder for every 0 <= m < 2^31: the same product exceeds m / n by less than 1, so the quotient is
// right or one too large.  For the rows of whole blocks (G * n_q of them: up to 2^24 with n up to 2^14).
LKV_HD int div_rem(int m, int n, uint32_t magic, int* rem) {
  int q = div_w(m, magic), r = m - q * n;
  if (r < 0) {
    --q;
    r += n;
  }
  *rem = r;
  return q;
}

// Row tiles and key ranges of attend_rows_kernel: m_rows = G * n_q rows per KV head in tiles of 32, cache_len cache rows,
// then s_t block keys of which query j sees those up to diag + j.
struct RowsShape {
  int m_rows, n_q;
  uint32_t nq_magic;
  int cache_len, s_t, diag;
};
// the end of the block keys that some row of tile t sees
LKV_HD int rows_tile_end(const RowsShape& s, int t) {
  if (s.s_t == 0) return 0;
  const int m0 = t * 32, m1 = (m0 + 32 < s.m_rows ? m0 + 32 : s.m_rows) - 1;
  int j0, j1;
  const int g0 = div_rem(m0, s.n_q, s.nq_magic, &j0), g1 = div_rem(m1, s.n_q, s.nq_magic, &j1);
  const int end = s.diag + (g0 == g1 ? j1 : s.n_q - 1) + 1, last = end < s.s_t ? end : s.s_t;
  return last > 0 ? last : 0;
}
// Row group pg (four pairs of tiles, the first and the last tile that remain each) cut into n_splits key ranges of equal
// time, which passes one key per unit where both waves of a pair work on their own tiles and two where they share one (the
// group's first pair stands for all): range r covers the units [r * share, (r + 1) * share), the first `both` of which are
// single keys, cache rows first.
struct RowsCut {
  int both, share, end;  // end: of the block keys that some row of the group sees
};
LKV_HD RowsCut rows_cut(const RowsShape& s, int pg, int n_splits) {
  const int n_tiles = (s.m_rows + 31) >> 5, n_pairs = (n_tiles + 1) >> 1, pr0 = pg * 4;
  const int ea = rows_tile_end(s, pr0), eb = rows_tile_end(s, n_tiles - 1 - pr0);
  const int lo = ea < eb ? ea : eb, hi = ea < eb ? eb : ea;
  RowsCut c;
  c.both = s.cache_len + lo;
  c.end = hi;
  for (int q = 1; q < 4; ++q)
    if (pr0 + q < n_pairs) {
      const int a = rows_tile_end(s, pr0 + q), b = rows_tile_end(s, n_tiles - 1 - pr0 - q);
      c.end = a > c.end ? a : c.end;
      c.end = b > c.end ? b : c.end;
    }
  const int total = c.both + (hi - lo + 1) / 2;
  c.share = ((total + n_splits - 1) / n_splits + 31) & ~31;
  return c;
}
// the cache rows of a group's last range, the fewest of all ranges
LKV_HD int rows_last_cache_range(const RowsShape& s, int pg, int n_splits) {
  const int64_t before = (int64_t)(n_splits - 1) * rows_cut(s, pg, n_splits).share;
  return before < s.cache_len ? (int)(s.cache_len - before) : 0;
}

}  // namespace lkv

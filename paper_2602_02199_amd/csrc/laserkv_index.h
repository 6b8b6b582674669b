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

}  // namespace lkv

// Row statistics shared by the layer's statistics kernel and the normaliser-only attention kernel: per query row the
// pair (reference, sum of 2^(x - reference)) over a range of keys, x the scaled logit.
#pragma once

#include "laserkv_device.h"

namespace lkv {

constexpr int RS_WAVES = 8;
constexpr int RS_THREADS = RS_WAVES * 64;

// keys per LDS chunk; two chunks fill 139 KiB
constexpr int row_stats_chunk(int row_bytes) { return row_bytes <= 256 ? 256 : 128; }
constexpr size_t row_stats_lds(int row_bytes) { return (size_t)2 * row_stats_chunk(row_bytes) * (row_bytes + 16); }

// Keys k_lo .. k_hi - 1 of the descriptor's rows against RT 32-row tiles per wave (q: the rows' MFMA fragments).  Waves
// that share rows take different 32-key tiles (ks, ks + wk, ...).  Keys are the A operand and rows the B operand, so a
// lane owns a row per tile; its two halves hold the same rows over different keys and are merged before the end.
// A row sees the keys below its lim[r]; every row sees the keys up to lim_all.  The reference is the maximum over the
// lane's first tile plus HEADROOM; complete tiles after it cost one fma, one exponential and one add per logit.  When a
// sum has grown past 1e34 after a chunk (a logit 137 above the first tile's, in powers of two; a thousand such sums can
// still be merged), the wave repeats that chunk from LDS with a reference that follows the maximum.  References are
// whole numbers, so that moving one rescales its sum exactly.
// What bounds it: matrix and vector work of a SIMD hardly overlap (16 matrix instructions of 32 clocks and 64 vector
// instructions of 4, 32 exponentials of 8 per pair of tiles).  512 rows over 63 520 keys of 8 heads 76 us = 870 TFLOP/s
// with the merge, a 128k layer 181 us = 800, 256 rows over 31 681 keys 28.6 us = 580 (start and merge are a third); a
// plain bf16 product reaches 1380.  64 rows per wave halve the LDS reads per instruction (32 rows: LDS-bound).
template <int DT, int D, int RT>
__device__ __forceinline__ void row_stats(uint4* smem, __amdgpu_buffer_rsrc_t ksrd, uint32_t kstride, int k_lo, int k_hi, int lim_all,
                                          const int (&lim)[RT], const uint4 (&q)[RT][D * (DT == DT_BF16 ? 2 : 4) / 32], float scale2,
                                          int ks, int wk, bool active, float (&ref)[RT], float (&sum)[RT]) {
  constexpr int CH = D * (DT == DT_BF16 ? 2 : 4) / 16, NCH = CH / 2, CHP = CH + 1;
  constexpr int KC = row_stats_chunk(CH * 16), TPC = KC / 32;
  constexpr int KL = KC * CH / RS_THREADS;
  constexpr int RPL = RS_THREADS / CH;
  const int tid = threadIdx.x, lane = tid & 63, rl = lane & 31, kg = lane >> 5;
  const uint32_t k_row = tid / CH, k_col = tid % CH;
  uint4 kpre[KL];
  auto prefetch = [&](int kc0) {
#pragma unroll
    for (int u = 0; u < KL; ++u) kpre[u] = buf_ld16(ksrd, (uint32_t)(kc0 + k_row + u * RPL) * kstride + k_col * 16);
  };
  auto store = [&](uint4* buf) {
#pragma unroll
    for (int u = 0; u < KL; ++u) buf[(k_row + u * RPL) * CHP + k_col] = kpre[u];
  };

#pragma unroll
  for (int r = 0; r < RT; ++r) {
    ref[r] = NEG_BIG;
    sum[r] = 0.0f;
  }
  bool first = true;  // no tile yet: the lane has no reference
  prefetch(k_lo);
  store(smem);
  lds_barrier();
  int cur = 0;
  for (int kc0 = k_lo; kc0 < k_hi; kc0 += KC) {
    const bool more = kc0 + KC < k_hi;
    if (more) prefetch(kc0 + KC);
    const uint4* sK = smem + (size_t)cur * KC * CHP;
    float kept[RT];
#pragma unroll
    for (int r = 0; r < RT; ++r) kept[r] = sum[r];
    bool fixed_ref = !first;  // wave-uniform
#pragma unroll 1
    for (int attempt = active ? 0 : 2; attempt < 2; ++attempt) {
#pragma unroll 1
      for (int nt = ks; nt < TPC; nt += wk) {
        const int kbase = kc0 + nt * 32;
        if (kbase >= k_hi) break;  // wave-uniform
        f32x16 acc[RT];
#pragma unroll
        for (int r = 0; r < RT; ++r)
#pragma unroll
          for (int e = 0; e < 16; ++e) acc[r][e] = 0.0f;
        const uint4* krow = sK + (size_t)(nt * 32 + rl) * CHP + kg;
#pragma unroll
        for (int i = 0; i < NCH; ++i) {
          const uint4 kf = krow[2 * i];
#pragma unroll
          for (int r = 0; r < RT; ++r) Mma<DT>::run(acc[r], kf, q[r][i]);
        }
        const bool whole = kbase + 32 <= k_hi && kbase + 31 <= lim_all;  // every row sees every key
        if (whole && fixed_ref) {
#pragma unroll
          for (int r = 0; r < RT; ++r)
#pragma unroll
            for (int e = 0; e < 16; ++e) sum[r] += fast_exp2(fmaf(acc[r][e], scale2, -ref[r]));
        } else {
#pragma unroll
          for (int r = 0; r < RT; ++r) {
            const int n_vis = whole ? 32 : min(k_hi, lim[r]) - kbase;
            if (acc_row(0, kg) < n_vis) {  // a lane that sees none of its keys keeps its state
              float mx = acc[r][0];
#pragma unroll
              for (int e = 1; e < 16; ++e) mx = acc_row(e, kg) < n_vis ? fmaxf(mx, acc[r][e]) : mx;
              const float nref = fmaxf(ref[r], ceilf(mx * scale2));  // scale2 > 0
              sum[r] *= fast_exp2(ref[r] - nref);
              ref[r] = nref;
#pragma unroll
              for (int e = 0; e < 16; ++e)
                sum[r] += acc_row(e, kg) < n_vis ? fast_exp2(fmaf(acc[r][e], scale2, -nref)) : 0.0f;
            }
          }
          if (first) {
            fixed_ref = true;
#pragma unroll
            for (int r = 0; r < RT; ++r) {
              ref[r] += HEADROOM;
              sum[r] = __builtin_amdgcn_ldexpf(sum[r], -(int)HEADROOM);
            }
          }
          first = false;
        }
      }
      // sums that have grown too large against the fixed reference: the chunk (still in LDS) once more, the reference
      // following the maximum
      bool over = false;
#pragma unroll
      for (int r = 0; r < RT; ++r) over |= !(sum[r] < 1.0e34f);
      if (attempt || !__any(over)) break;
      fixed_ref = false;
#pragma unroll
      for (int r = 0; r < RT; ++r) {
        const float nref = kept[r] > 1.0e10f ? ref[r] + ceilf(fast_log2(kept[r])) : ref[r];
        sum[r] = kept[r] * fast_exp2(ref[r] - nref);
        ref[r] = nref;
      }
    }
    if (more) store(smem + (size_t)(cur ^ 1) * KC * CHP);
    cur ^= 1;
    lds_barrier();
  }
#pragma unroll
  for (int r = 0; r < RT; ++r) lse_merge(ref[r], sum[r], half_other(ref[r], kg), half_other(sum[r], kg));
}

}  // namespace lkv

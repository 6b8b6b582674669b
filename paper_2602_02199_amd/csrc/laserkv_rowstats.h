// Row statistics shared by the layer's statistics kernel and the normaliser-only attention kernel: per query row the
// pair (reference, sum of 2^(x - reference)) over a range of keys, x the scaled logit.
#pragma once

#include "laserkv_device.h"

namespace lkv {

constexpr int RS_WAVES = 8;
constexpr int RS_THREADS = RS_WAVES * 64;

// Keys stand in a ring of LDS stages as the asynchronous loads leave them: 1024 bytes at a time, which is RPG rows, PAD
// bytes between two such groups.  Chunk c of row r lies at position c ^ (r % RPG) of its row: eight consecutive rows then
// hold one chunk in eight different sets of banks, and a lane's operand chunks are RPG / 2 addresses plus constants (with
// rows permuted as a whole every chunk of a row has an address of its own, an addition each per tile).
template <int CH>  // 16-byte chunks per row
struct KeyRing {
  static constexpr int RPG = 64 / CH;
  static constexpr int PAD = RPG < 8 ? RPG * 16 : 0;
  static constexpr int GROUP = 1024 + PAD;
  static constexpr int TILE = 32 / RPG * GROUP;      // bytes of 32 keys
  static constexpr int KC = CH <= 16 ? 128 : 64;     // keys per stage
  static constexpr int STAGE = KC / 32 * TILE;
  static constexpr int STAGES = 4;
  static constexpr int NA = RPG > 2 ? RPG / 2 : 1;   // different addresses of a lane's operand chunks
};
constexpr size_t row_stats_lds(int row_bytes) {
  return row_bytes <= 128 ? (size_t)KeyRing<8>::STAGES * KeyRing<8>::STAGE
         : row_bytes <= 256 ? (size_t)KeyRing<16>::STAGES * KeyRing<16>::STAGE : (size_t)KeyRing<32>::STAGES * KeyRing<32>::STAGE;
}

// Whether ranges of this many keys take the instance for long ones: from twelve chunks on (512 rows over 63 520 keys in ranges
// of 15.5 chunks 77.1 -> 73.5 us, 64k layer of 18 a range 167.9 -> 166.6; 256 rows in ranges of 8 29.1 -> 29.6, 16k layer of 5
// a range 59.3 -> 60.4).
constexpr bool row_stats_long(int dtype, int row_bytes, int rt, int keys) {
  return dtype == DT_BF16 && rt == 2 && keys >= 12 * (row_bytes <= 256 ? 128 : 64);
}

// Keys k_lo .. k_hi - 1 of the descriptor's rows against RT 32-row tiles per wave (q: the rows' MFMA fragments).  Waves
// that share rows take different 32-key tiles (ks, ks + wk, ...; active, ks and wk are the same in all lanes of a wave).
// Keys are the A operand and rows the B operand, so a lane owns a row per tile; its two halves hold the same rows over
// different keys and are merged before the end.
// A row sees the keys below its lim[r]; every row sees the keys up to lim_all.  The reference is the maximum over the
// lane's first tile plus HEADROOM; complete tiles after it cost one fma, one exponential and one add per logit.  When a
// tile lifts a sum past 1e34 (a logit 137 above the first tile's, in powers of two; a thousand such sums can still be
// merged), it is added again, its logits being in registers still, with a reference that follows the maximum.  References
// are whole numbers, so that moving one rescales its sum exactly.
// The products of a tile and the exponentials of the tile before it are independent: they are issued alternately, four
// vector instructions and two exponentials (40 clocks of the vector unit, issue of the matrix instruction included) beside
// every matrix instruction (32 clocks of the matrix unit).  Loads run two to three chunks ahead, so that one barrier per
// chunk publishes what has landed and frees the stage before it; the tiles of a wave run on across it.
// What bounds it: at a full clock the vector unit; over a whole layer the clock, which power sets (the same launch takes
// 180 us on random keys from HBM, 138 when they come from the caches, 116 when they are zeros).  512 rows over 63 520 keys
// of 8 heads, 128k layer of 256 groups: 172-181 -> 154-160 us = 910-940 TFLOP/s; 256 rows over 31 681 keys 28.4-30 ->
// 25.4-27 us.  Before: one tile after another, products, then exponentials; the first product of every chunk waited for the
// next chunk's loads.  Barriers cost: chunks of 64 keys (eight stages) 174 us, of 256 (two stages, the pipeline drained at
// each) 161.  64 rows per wave halve the LDS reads per instruction (32 rows: LDS-bound).
// LONG: whole chunks in the middle of a range take a loop without control per tile (see middle_chunks).
template <int DT, int D, int RT, bool LONG>
__device__ __forceinline__ void row_stats(uint4* smem, srd_words ksrd, uint32_t kstride, int k_lo, int k_hi, int lim_all,
                                          const int (&lim)[RT], uint4 (&q)[RT][D * (DT == DT_BF16 ? 2 : 4) / 32], float scale2,
                                          int ks, int wk, bool active, float (&ref)[RT], float (&sum)[RT]) {
  constexpr int CH = D * (DT == DT_BF16 ? 2 : 4) / 16, NCH = CH / 2;
  using L = KeyRing<CH>;
  constexpr int KC = L::KC, TPC = KC / 32, S = L::STAGES;
  // Waves that bring the keys in.  In long ranges the first wave of every SIMD: the address unit takes some five hundred clocks
  // for a chunk, and the second waves have the SIMDs to themselves meanwhile (512 rows over 63 520 keys 70.0 -> 68.1 us, 128k
  // layer 477.6 -> 476.6).  In short ranges all of them, the first keys are there sooner (256 rows over 31 681 keys 28.15 us, 28.4
  // with half of them; over 74 keys 9.6, 9.7).  In fp32, whose tiles take several times as long, the first ones always: dimension
  // 128, 32 rows a head over 9000 keys 29.2 -> 28.3, over 4000 17.5 -> 17.2, short ranges the same (over 64, 500 and 2000 keys 10.3,
  // 10.9 and 13.1 with all waves, 10.4, 11.0 and 13.1).
  constexpr int LOADERS = LONG || DT == DT_F32 ? RS_WAVES / 2 : RS_WAVES;
  constexpr int LOADS = KC * CH / (LOADERS * 64);  // each, per stage
  // registers for a second tile's logits (in fp32 matrix instructions take nearly all of the time: twice the code is slower)
  constexpr bool PIPED = DT == DT_BF16 && RT * NCH <= 16;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, rl = lane & 31, kg = lane >> 5;
  const int n_keys = k_hi - k_lo;
  const int n_tiles = (n_keys + 31) >> 5, n_chunks = (n_keys + KC - 1) / KC;
  const int n_whole = max(min(k_hi, lim_all + 1) - k_lo, 0) >> 5;  // tiles of which every row sees every key

  // Waves that share rows work on wk consecutive tiles at a time.  Chunks are opened `span` at once, so that these tiles are
  // there together: with a barrier between them, eight waves on four tiles each ran one half after the other (32 rows over
  // 9000 keys, bf16 9.8 -> 9.4 us, fp32 23.6 -> 18.1).
  if (wk > 2 * TPC) {
    wk = 2 * TPC;
    active = active && ks < wk;
  }
  const int span = wk > TPC ? 2 : 1;
  const bool roll = PIPED && span == 1;  // the next tile's keys, one chunk on at most, are read while the current ones are multiplied
  const int ahead = roll ? 1 : 0;

  const uint32_t lds0 = lds_offset(smem);
  // loads: wave w brings the w-th of every LOADERS groups of a stage
  const uint32_t ld_row = lane / CH, ld_col = ((lane % CH) ^ (ld_row % L::RPG)) * 16;
  const uint32_t ld_off = ld_row * kstride + ld_col;
  auto prefetch = [&](int c) {
    if (LOADERS < RS_WAVES && wave >= LOADERS) return;
    const int row = c * KC + wave * L::RPG;  // of the range: the first group's first
    uint32_t dst = lds0 + (c % S) * L::STAGE + wave * L::GROUP;
    if ((c + 1) * KC <= n_keys) {
      uint32_t src = (uint32_t)(k_lo + row) * kstride;
#pragma unroll
      for (int u = 0; u < LOADS; ++u, src += LOADERS * L::RPG * kstride, dst += LOADERS * L::GROUP) async_ld16(ksrd, ld_off, src, dst);
    } else if (c < n_chunks) {
      // Rows past the end repeat the last one.  Where everything is waited for at the start, only whole tiles are loaded (256
      // rows over 74 keys 9.5 -> 9.35 us); else every chunk has as many loads as `await` counts.
      const int n_loads = n_chunks <= span + ahead ? min((n_tiles * 32 - row + LOADERS * L::RPG - 1) / (LOADERS * L::RPG), LOADS) : LOADS;
#pragma unroll 1
      for (int u = 0; u < n_loads; ++u, dst += LOADERS * L::GROUP)
        async_ld16(ksrd, (uint32_t)(k_lo + min(row + u * LOADERS * L::RPG + (int)ld_row, n_keys - 1)) * kstride + ld_col, 0u, dst);
    }
  };
  int open = span - 1, issued = min(span + ahead, n_chunks);
  auto await = [&](int c) {  // chunks up to c
    static_assert(S == 4, "at most two chunks are on their way behind the one waited for");
    const int flying = issued - 1 - c;
    if (flying >= 2) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * LOADS) : "memory");
    else if (flying == 1) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(LOADS) : "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  };
  // Opens chunk c with those of its span: they (and the one behind them) have landed for every wave, and every wave has left
  // the span before, whose stages take the next loads.
  auto open_to = [&](int c) {
    while (open < c) {
      ++open;
      if (span == 1 || !(open & 1)) {
        await(min(open + span - 1 + ahead, n_chunks - 1));
        lds_barrier();
      }
      prefetch(open + S - span);
      issued = min(open + S - span + 1, n_chunks);
    }
  };

  // LDS addresses of the lane's row in tile 0: chunk 2i + kg is at at[i % NA] + i / NA * (NA * 32)
  uint32_t at[L::NA];
#pragma unroll
  for (int i = 0; i < L::NA; ++i) at[i] = lds0 + rl / L::RPG * L::GROUP + rl % L::RPG * (CH * 16) + (((2 * i + kg) ^ (rl % L::RPG)) * 16);
  uint4 kf[NCH];
  auto tile_off = [&](int t) -> uint32_t { return (uint32_t)(t / TPC % S) * L::STAGE + (uint32_t)(t % TPC) * L::TILE; };
  uint32_t from[L::NA];  // the lane's addresses in the tile that is read
  auto read_from = [&](int t) {
#pragma unroll
    for (int i = 0; i < L::NA; ++i) from[i] = opaque(at[i] + tile_off(t));
  };
  auto load = [&](int i) { kf[i] = lds_ld16(from[i % L::NA], i / L::NA * (L::NA * 32)); };

  // the first chunks' loads, then the rows that the caller has on their way, then the other chunks': the wait for the rows
  // covers all loads issued before it
#pragma unroll 1
  for (int c = 0; c < span + ahead; ++c) prefetch(c);
#pragma unroll
  for (int r = 0; r < RT; ++r) {
    ref[r] = NEG_BIG;
    sum[r] = 0.0f;
#pragma unroll
    for (int i = 0; i < NCH; ++i) landed(q[r][i]);
  }
  async_wait();
  lds_barrier();
#pragma unroll 1
  for (int c = span + ahead; c < S; ++c) prefetch(c);
  issued = min(S, n_chunks);

  bool first = true;      // no tile yet: the lane has no reference
  // one tile's logits, the reference following the maximum
  auto careful = [&](const f32x16 (&acc)[RT], int t) {
#pragma unroll
    for (int r = 0; r < RT; ++r) {
      const int n_vis = t < n_whole ? 32 : min(k_hi, lim[r]) - (k_lo + t * 32);
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
#pragma unroll
      for (int r = 0; r < RT; ++r) {
        ref[r] += HEADROOM;
        sum[r] = __builtin_amdgcn_ldexpf(sum[r], -(int)HEADROOM);
      }
    }
    first = false;
  };
  float kept[RT];
  // sums that have grown too large: the tile once more, from the sums before it
  auto check = [&](const f32x16 (&acc)[RT], int t) {
    bool over = false;
#pragma unroll
    for (int r = 0; r < RT; ++r) over |= !(sum[r] < 1.0e34f);
    if (!__any(over)) return;
#pragma unroll
    for (int r = 0; r < RT; ++r) {
      const float nref = kept[r] > 1.0e10f ? ref[r] + ceilf(fast_log2(kept[r])) : ref[r];
      sum[r] = kept[r] * fast_exp2(ref[r] - nref);
      ref[r] = nref;
    }
    careful(acc, t);
  };
  auto add = [&](const f32x16 (&acc)[RT]) {
#pragma unroll
    for (int r = 0; r < RT; ++r) kept[r] = sum[r];
#pragma unroll
    for (int e = 0; e < 16; ++e)
#pragma unroll
      for (int r = 0; r < RT; ++r) sum[r] += fast_exp2(fmaf(acc[r][e], scale2, -ref[r]));
  };
  int t = active ? ks : n_tiles, pending = -1;
  bool here = false;                    // kf holds tile t
  // the products of tile t, and what the tile before it still has to add
  auto fire = [&](f32x16 (&next)[RT], const f32x16 (&done)[RT]) {
    open_to(t / TPC | (span - 1));
    if (!here) {
      read_from(t);
#pragma unroll
      for (int i = 0; i < NCH; ++i) load(i);
    }
    here = roll;
    read_from(roll && t + wk < n_tiles ? t + wk : t);
    const bool fast = pending >= 0 && pending < n_whole && !first;  // wave-uniform
    auto products = [&]() {
#pragma unroll
      for (int r = 0; r < RT; ++r)
#pragma unroll
        for (int e = 0; e < 16; ++e) next[r][e] = 0.0f;
#pragma unroll
      for (int i = 0; i < NCH; ++i) {
#pragma unroll
        for (int r = 0; r < RT; ++r) Mma<DT>::run(next[r], kf[i], q[r][i]);
        load(i);
      }
    };
    if (fast) {
      products();
      add(done);
      if (DT == DT_BF16) {
#pragma unroll
        for (int i = 0; i < NCH; ++i) {
#pragma unroll
          for (int r = 0; r < RT; ++r) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);         // a matrix instruction
            __builtin_amdgcn_sched_group_barrier(0x002, 32 / NCH, 0);  // vector instructions beside it
            __builtin_amdgcn_sched_group_barrier(0x400, 16 / NCH, 0);  // exponentials
          }
          __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);           // a read from LDS
        }
      }
      check(done, pending);
    } else {
      products();
      if (pending >= 0) careful(done, pending);
    }
    pending = t;
    t += wk;
  };
  auto drain = [&](const f32x16 (&done)[RT]) {
    if (pending < 0) return;
    if (pending < n_whole && !first) {
      add(done);
      check(done, pending);
    } else {
      careful(done, pending);
    }
  };
  f32x16 acc0[RT], acc1[RT];
  // A tile in the middle of a range: its products beside the exponentials of the tile before, in a fixed order.  What stands
  // between two fences is issued beside one matrix instruction: exponents one step ahead of their exponentials, sums one behind.
  auto middle = [&](f32x16 (&next)[RT], const f32x16 (&done)[RT]) {
    constexpr int SLOTS = NCH * RT, PER = 16 * RT / SLOTS;  // matrix instructions, logits beside each
#pragma unroll
    for (int r = 0; r < RT; ++r) {
      kept[r] = sum[r];
#pragma unroll
      for (int e = 0; e < 16; ++e) next[r][e] = 0.0f;
    }
    float x[PER], y[PER];
    auto exponents = [&](int j) {
#pragma unroll
      for (int k = 0; k < PER; ++k) x[k] = fmaf(done[(j * PER + k) % RT][(j * PER + k) / RT], scale2, -ref[(j * PER + k) % RT]);
    };
    auto sums = [&](int j) {
#pragma unroll
      for (int k = 0; k < PER; ++k) sum[(j * PER + k) % RT] += y[k];
    };
    exponents(0);
#pragma unroll
    for (int j = 0; j < SLOTS; ++j) {
      Mma<DT>::run(next[j % RT], kf[j / RT], q[j % RT][j / RT]);
      if (j % RT == RT - 1) load(j / RT);
      if (j > 0) sums(j - 1);
#pragma unroll
      for (int k = 0; k < PER; ++k) y[k] = fast_exp2(x[k]);
      if (j + 1 < SLOTS) exponents(j + 1);
      __builtin_amdgcn_sched_barrier(0);
    }
    sums(SLOTS - 1);
    check(done, pending);
    pending = t;
    t += wk;
  };
  // Chunks in the middle of a range, from one that is not open yet on: every row sees every key, the loads that opening them
  // starts are whole chunks, and each has an even number of tiles for the wave.  Between the barriers there is no control flow
  // but the test for sums that have grown too large (128k layer 157 -> 149 us, groups of eight 149.6 -> 141.7).  An instance of
  // its own, for long ranges: the code alone made short ones 1-4 % slower.
  auto middle_chunks = [&]() {
    if (wk > 2 || !roll || !here || first || pending < 0 || pending >= n_whole || t / TPC <= open) return;
    while ((open + 1 + S) * KC <= n_keys && (open + 2) * TPC <= n_whole) {
      asm volatile("s_waitcnt vmcnt(%0)" ::"n"(LOADS) : "memory");
      lds_barrier();
      ++open;
      prefetch(open + S - 1);
      issued = open + S;
      const uint32_t step = (uint32_t)wk * L::TILE;
      uint32_t off = (uint32_t)(open % S) * L::STAGE + (uint32_t)ks * L::TILE;
      const uint32_t off_next = (uint32_t)((open + 1) % S) * L::STAGE + (uint32_t)ks * L::TILE;
      for (int u = TPC / wk; u > 0; u -= 2) {
        off += step;
#pragma unroll
        for (int i = 0; i < L::NA; ++i) from[i] = opaque(at[i] + off);
        middle(acc0, acc1);
        off = u > 2 ? off + step : off_next;
#pragma unroll
        for (int i = 0; i < L::NA; ++i) from[i] = opaque(at[i] + off);
        middle(acc1, acc0);
      }
    }
  };
  if (PIPED) {
    const bool even = wave < RS_WAVES / 2;  // the two waves of a SIMD take turns at being served first
#pragma unroll 1
    for (;;) {
      if (LONG) middle_chunks();
      if (t >= n_tiles) {
        drain(acc1);
        break;
      }
      even ? __builtin_amdgcn_s_setprio(1) : __builtin_amdgcn_s_setprio(0);
      fire(acc0, acc1);
      if (t >= n_tiles) {
        drain(acc0);
        break;
      }
      even ? __builtin_amdgcn_s_setprio(0) : __builtin_amdgcn_s_setprio(1);
      fire(acc1, acc0);
    }
    __builtin_amdgcn_s_setprio(0);
  } else {
#pragma unroll 1
    for (; t < n_tiles; t += wk) {
      open_to(t / TPC | (span - 1));
      read_from(t);
#pragma unroll
      for (int r = 0; r < RT; ++r)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc0[r][e] = 0.0f;
#pragma unroll
      for (int i = 0; i < NCH; ++i) {
        load(i);
#pragma unroll
        for (int r = 0; r < RT; ++r) Mma<DT>::run(acc0[r], kf[i], q[r][i]);
      }
      pending = t;
      drain(acc0);
    }
  }
  open_to((n_chunks - 1) | (span - 1));
  async_wait();
  lds_barrier();  // every wave has left the stages
#pragma unroll
  for (int r = 0; r < RT; ++r) lse_merge(ref[r], sum[r], half_other(ref[r], kg), half_other(sum[r], kg));
}

}  // namespace lkv

// A layer whose blocks are all in memory, compressed with a few launches for all of its blocks together
// (laserkv_compress_layer).  The blocks of a layer do not depend on each other: the look-back keys of block t are
// the local window of block t - 1 (Sec. 3.2), which is always kept, so they are simply the rows in front of the
// block in the layer's own key tensor.  Every (block, KV head) pair is one independent group of work; with a layer's
// worth of groups in a launch the chip is full, and what a launch per block pays once per block (launch, loads of the
// window rows and hyperplanes, tail) is paid once per layer.
//
//   layer_stats_kernel   per window row, partial (reference, sum) of 2^(logit) over a key range (Alg. 1 step 3); then SimHash
//                        codes of the window rows (Sec. 3.3 "Recall") and their histograms, compact enough for the score
//                        kernel's LDS                                                                         [MFMA]
//   layer_codes_kernel   the codes alone, where the caller brings the statistics                              [MFMA]
//   layer_score_kernel   one pass over the block's keys: pooled probabilities (Alg. 1 step 3), sign bits against all
//                        hyperplanes, collision counts (Alg. 1 step 6)                                        [MFMA]
//   then the select + append kernel of laserkv_kernels.hip over all groups.
//
// In both sweeps the window rows stay in registers for the whole key range (two 32-row tiles per wave, so a key
// fragment read from LDS feeds two matrix instructions) and the keys stream through LDS stages, one barrier per chunk: the
// statistics through four stages, the scores through two, both filled by asynchronous loads.
#include "laserkv_device.h"
#include "laserkv_kernels.h"
#include "laserkv_rowstats.h"

#include <limits.h>

#include <type_traits>

namespace lkv {

constexpr int LY_WAVES = 8;
constexpr int LY_THREADS = LY_WAVES * 64;
constexpr int LY_ROWS = 512;         // window rows per group at most
constexpr int LY_KC = 128;           // keys per LDS chunk of the score kernel
constexpr int LY_HEAVY = 36;         // words per table's list of heavy bins: at most LY_ROWS / 15 = 34 of them
constexpr int LY_CODE_PLANES = 256;  // hyperplanes per pass of layer_codes_kernel at most

// Rows of LDS for the hyperplanes of a set of tables: a wave's tiles of 32 may start at any table and end past the last one
constexpr int code_plane_rows(int tables, int n_bits) { return tables * n_bits + 31; }

struct LayerGroup {
  int g, b, h, lo, s_t, n_ctx;
};
__device__ __forceinline__ LayerGroup layer_group(const LayerParams& p, int g) {
  LayerGroup r;
  r.g = g;
  r.b = g / p.n_kv_heads;
  r.h = g - r.b * p.n_kv_heads;
  r.lo = r.b * p.s_block;
  r.s_t = min(p.s_block, p.n_tok - r.lo);
  r.n_ctx = r.b ? p.n_ctx : 0;
  return r;
}

__device__ __forceinline__ const char* layer_row(const LayerParams& p, const LayerGroup& gr, int m) {
  const int g = div_w(m, p.w_magic), j = m - g * p.w;
  return p.q.base + gr.b * p.q_stride_block + (int64_t)(gr.h * p.group + g) * p.q.stride_head + (int64_t)j * p.q.stride_row;
}

// ---------------------------------------------------------------------------------------------
// Codes of a group's window rows.  Waves hold 32 or 64 rows as MFMA operands and the tables
// pass by in sets whose hyperplanes and histograms fit the LDS.  A set's codes are counted in LDS histograms (16-bit
// bins, 32 bins per 17 words against bank conflicts), which leave as cells of 16, 8 or 4 bits per bin, the widest with
// which a group's tables fit 64 KiB of the score kernel's LDS (4 bits at K = 12, L = 32).  A narrow cell that is full
// stands for a count the table's list of heavy bins holds: (code << 16 | count) each, their number in front.
// Codes wider than 12 bits: the codes themselves are stored (count_kernel does the counting).
// ---------------------------------------------------------------------------------------------
constexpr int LY_CODE_THREADS = 1024;

// b: the wave's rows row0 .. as MFMA fragments; t_first, t_step: the workgroup's sets of `n_set` tables.  Waves that share rows
// (wk of them) take different tables of a set.  All NT threads take part.
template <int DT, int D, int RT, int NT>
__device__ __forceinline__ void window_codes(const LayerParams& p, int g, uint4* smem, const uint4 (&b)[RT][D * (DT == DT_BF16 ? 2 : 4) / 32],
                                             int row0, bool active, int ks, int wk, int n_set, int t_first, int t_step) {
  constexpr int ES = DT == DT_BF16 ? 2 : 4;
  constexpr int CH = D * ES / 16, NCH = CH / 2, CHP = CH + 1;
  constexpr int NPL = LY_CODE_PLANES * CH / NT;  // 16-byte pieces of hyperplanes per thread at most
  typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
  const int tid = threadIdx.x, lane = tid & 63, rl = lane & 31, kg = lane >> 5;
  const bool wide = p.cells == nullptr;
  const int words = (1 << p.n_bits) >= 32 ? (1 << p.n_bits) >> 5 : 1;  // groups of 32 bins per table
  const int hp = words * 17;

  uint4* sP = smem;                                                                          // [planes of a set][CHP]
  uint32_t* sH = reinterpret_cast<uint32_t*>(smem + (size_t)code_plane_rows(n_set, p.n_bits) * CHP);  // [n_set][hp]
  int* sHeavy = reinterpret_cast<int*>(sH + ((n_set * hp + 3) & ~3));                        // [n_set]

  uint4 pre[NPL];  // the next set's hyperplanes, on their way while the current set is worked on
  auto fetch = [&](int t0) {
    const int np = min(n_set, p.n_tables - t0) * p.n_bits;
#pragma unroll
    for (int u = 0; u < NPL; ++u) {
      const int row = (tid + u * NT) / CH;
      if (row < np) pre[u] = ld16(p.planes + (size_t)(t0 * p.n_bits + row) * (D * ES) + tid % CH * 16);
    }
  };
  if (t_first < p.n_tables) fetch(t_first);
  const uint32_t code_mask = (1u << p.n_bits) - 1u;
  const int cbits = 32 >> p.cell_log, cw_log = max(p.n_bits - p.cell_log, 0);  // cell_words = 1 << cw_log
  const uint32_t cmax = cbits == 16 ? 0xffffu : (1u << cbits) - 1u;
  for (int t0 = t_first; t0 < p.n_tables; t0 += t_step) {
    const int n_tab = min(n_set, p.n_tables - t0), np = n_tab * p.n_bits;
    __syncthreads();  // the previous set's histograms have been read
#pragma unroll
    for (int u = 0; u < NPL; ++u) {
      const int r = (tid + u * NT) / CH;
      if (r < np) sP[r * CHP + tid % CH] = pre[u];
    }
    if (!wide) {
      uint4* h4 = reinterpret_cast<uint4*>(sH);
      for (int i = tid; i < (n_tab * hp + 3) / 4; i += NT) h4[i] = make_uint4(0u, 0u, 0u, 0u);
      if (tid < n_tab) sHeavy[tid] = 0;
    }
    __syncthreads();
    if (t0 + t_step < p.n_tables) fetch(t0 + t_step);
    const int ta = n_tab * ks / wk, tb = n_tab * (ks + 1) / wk;  // this wave's tables of the set
    // Codes of 16 bits lie in sig_q as the tiles' words follow each other: eight at a time go out (two bytes at a time every
    // store writes to 64 lines)
    const bool plain = wide && p.n_bits == 16 && ((p.n_tables | (t0 + ta)) & 7) == 0;
    if (active && ta < tb) {
      uint32_t prev[RT] = {};
      uint4 last4[RT];  // the last four words
      int tt0 = ta;  // first table whose bits are not complete yet
#pragma unroll 1
      for (int t = 0; tt0 < tb; ++t) {
        const uint4* prow = sP + (size_t)(ta * p.n_bits + t * 32 + plane_row(rl)) * CHP + kg;  // rows past the set's planes hold anything
        f32x16 acc[RT];
#pragma unroll
        for (int r = 0; r < RT; ++r)
#pragma unroll
          for (int e = 0; e < 16; ++e) acc[r][e] = 0.0f;
#pragma unroll
        for (int i = 0; i < NCH; ++i) {
          const uint4 pf = prow[2 * i];
#pragma unroll
          for (int r = 0; r < RT; ++r) Mma<DT>::run(acc[r], pf, b[r][i]);
        }
        const int tt1 = min(ta + 32 * (t + 1) / p.n_bits, tb);  // tables complete after this tile
#pragma unroll
        for (int r = 0; r < RT; ++r) {
          uint32_t neg = 0u;
#pragma unroll
          for (int e = 15; e >= 0; --e) neg = __builtin_amdgcn_alignbit(neg, __float_as_uint(acc[r][e]), 31);
          const uint32_t pos = ~neg & 0xffffu;  // bit = projection >= 0
          const uint32_t other = half_other(pos, kg);
          const uint32_t word = kg ? (other | (pos << 16)) : (pos | (other << 16));
          const int row = row0 + r * 32 + rl;
          last4[r] = make_uint4(last4[r].y, last4[r].z, last4[r].w, word);
          if (plain && ta + 2 * (t | 3) + 1 < tb) {
            if ((t & 3) == 3 && row < p.m_rows && kg == (r & 1)) *reinterpret_cast<uint4*>(p.sig_q + ((size_t)g * p.m_rows + row) * p.n_tables + t0 + ta + 2 * (t - 3)) = last4[r];
          } else if (row < p.m_rows)
            for (int tt = tt0 + ((tt0 ^ kg) & 1); tt < tt1; tt += 2) {  // tables alternate between the two lanes of a row
              const int at = (tt - ta) * p.n_bits - 32 * t;  // its first bit in this tile's word, below 0: in the word before
              const uint32_t code = __builtin_amdgcn_alignbit(word, at < 0 ? prev[r] : word, at & 31) & code_mask;
              if (wide) p.sig_q[((size_t)g * p.m_rows + row) * p.n_tables + t0 + tt] = (uint16_t)code;
              else atomicAdd(sH + tt * hp + (code >> 5) * 17 + ((code & 31u) >> 1), 1u << ((code & 1u) * 16));
            }
          prev[r] = word;
        }
        tt0 = tt1;
      }
    }
    if (wide) continue;
    __syncthreads();
    // cells of CPW per word, WORDS words at a time: two bins at a time, clamped and moved next to each other
    auto pack = [&](auto cpw, auto n_words) {
      constexpr int CPW = decltype(cpw)::value, CB = 32 / CPW, WORDS = decltype(n_words)::value;
      const int per_log = cw_log - (WORDS == 4 ? 2 : 0);
      for (int i = tid; i < n_tab << per_log; i += NT) {
        const int tt = i >> per_log, cw = (i & ((1 << per_log) - 1)) * WORDS, c0 = cw * CPW;
        const uint32_t* hist = sH + tt * hp + (c0 >> 5) * 17 + ((c0 & 31) >> 1);  // at most 32 bins, within their 17 words
        const size_t table = (size_t)g * p.n_tables + t0 + tt;
        uint32_t out[4] = {0u, 0u, 0u, 0u};
        u16x2 most = {0, 0};
#pragma unroll
        for (int u = 0; u < WORDS * CPW / 2; ++u) {
          const u16x2 v = __builtin_bit_cast(u16x2, hist[u]), limit = {(unsigned short)cmax, (unsigned short)cmax};
          most = __builtin_elementwise_max(most, v);
          const uint32_t two = __builtin_bit_cast(uint32_t, __builtin_elementwise_min(v, limit));
          out[u / (CPW / 2)] |= (CPW == 2 ? two : (two | two >> (16 - CB)) & ((1u << (2 * CB & 31)) - 1u)) << (2 * CB * u & 31);
        }
        uint32_t* dst = p.cells + table * p.cell_words + cw;
        if (WORDS == 4) *reinterpret_cast<uint4*>(dst) = make_uint4(out[0], out[1], out[2], out[3]);
        else *dst = out[0];
        if (max(most.x, most.y) >= cmax)
          for (int u = 0; u < WORDS * CPW; ++u) {
            const uint32_t c = hist[u >> 1] >> ((u & 1) * 16) & 0xffffu;
            if (c >= cmax) p.heavy[table * LY_HEAVY + 1 + atomicAdd(&sHeavy[tt], 1)] = (uint32_t)(c0 + u) << 16 | c;
          }
      }
    };
    auto pack_cells = [&](auto cpw) {
      if (cw_log >= 2) pack(cpw, std::integral_constant<int, 4>{});
      else pack(cpw, std::integral_constant<int, 1>{});
    };
    if (p.cell_log == 1) pack_cells(std::integral_constant<int, 2>{});
    else if (p.cell_log == 2) pack_cells(std::integral_constant<int, 4>{});
    else pack_cells(std::integral_constant<int, 8>{});
    __syncthreads();
    if (tid < n_tab) p.heavy[((size_t)g * p.n_tables + t0 + tid) * LY_HEAVY] = (uint32_t)sHeavy[tid];
  }
}

template <int DT, int D>
__global__ __launch_bounds__(LY_CODE_THREADS) void layer_codes_kernel(LayerParams p) {
  constexpr int NCH = D * (DT == DT_BF16 ? 2 : 4) / 32;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, rl = lane & 31, kg = lane >> 5;
  const LayerGroup gr = layer_group(p, blockIdx.x);
  extern __shared__ uint4 smem[];
  uint4 b[1][NCH];  // this wave's 32 window rows
  const bool active = wave * 32 < p.m_rows;
  if (active) {
    const char* ptr = layer_row(p, gr, min(wave * 32 + rl, p.m_rows - 1));
#pragma unroll
    for (int i = 0; i < NCH; ++i) b[0][i] = ld16(ptr + (2 * i + kg) * 16);
  }
  window_codes<DT, D, 1, LY_CODE_THREADS>(p, gr.g, smem, b, wave * 32, active, 0, 1, p.code_tables, blockIdx.y * p.code_tables, gridDim.y * p.code_tables);
}

// ---------------------------------------------------------------------------------------------
// Row statistics (laserkv_rowstats.h).  Workgroup = (group, key range); 2^wr_log waves share the rows (RT tiles each) and,
// where the rows need fewer than eight waves, the others take different key tiles.
// The rows' codes follow, while the rows are in registers: a launch of their own paid its start, the rows' way into registers
// and a round of workgroups once more (16k layer 7.0 + 21.2 -> 23.4 us, 64k 13.8 + 50.9 -> 59.7, groups of eight 15.1 + 144.7
// -> 157.7, 128k 33.7 + 155.6 -> 186).
// ---------------------------------------------------------------------------------------------
template <int DT, int D, int RT, bool LONG>
__global__ __launch_bounds__(LY_THREADS) void layer_stats_kernel(LayerParams p) {
  constexpr int NCH = D * (DT == DT_BF16 ? 2 : 4) / 32;
  static_assert(LY_THREADS == RS_THREADS, "row_stats works with eight waves");
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, rl = lane & 31, kg = lane >> 5;
  const int lin = xcd_major(blockIdx.x, gridDim.x);
  const int sp = lin % p.stat_splits;
  const LayerGroup gr = layer_group(p, lin / p.stat_splits);
  const int wk = LY_WAVES >> p.wr_log;                     // waves over different key tiles
  const int wi = wave & ((1 << p.wr_log) - 1), ks = wave >> p.wr_log;
  const int row0 = wi * RT * 32;
  const bool active = row0 < p.m_rows;
  const int n_keys = gr.n_ctx + gr.s_t;                    // look-back keys first
  const int k_lo = min(sp * p.stat_keys, n_keys), k_hi = min(k_lo + p.stat_keys, n_keys);
  const int lim0 = gr.n_ctx + gr.s_t - p.w;                // key k is visible to window row j iff k <= lim0 + j

  extern __shared__ uint4 smem[];

  uint4 q[RT][NCH];
  int lim[RT];
#pragma unroll
  for (int r = 0; r < RT; ++r) {
    const int m = min(row0 + r * 32 + rl, p.m_rows - 1);
    lim[r] = lim0 + m - div_w(m, p.w_magic) * p.w + 1;     // end of the visible keys
    const char* ptr = layer_row(p, gr, m);
#pragma unroll
    for (int i = 0; i < NCH; ++i) q[r][i] = ld16(ptr + (2 * i + kg) * 16);
  }
  const uint32_t kstride = (uint32_t)p.k.stride_row;
  const srd_words ksrd = make_srd_words(p.k.base + (int64_t)gr.h * p.k.stride_head + (int64_t)(gr.lo - gr.n_ctx) * p.k.stride_row,
                                        (uint32_t)n_keys * kstride);
  float ref[RT], sum[RT];
  row_stats<DT, D, RT, LONG>(smem, ksrd, kstride, k_lo, k_hi, lim0, lim, q, p.scale2, ks, wk, active, ref, sum);
  if (active)
#pragma unroll
    for (int r = 0; r < RT; ++r) {
      const int row = row0 + r * 32 + rl;
      if (kg == 0 && row < p.m_rows)
        p.part[((size_t)gr.g * p.m_rows + row) * p.n_parts + sp * wk + ks] = make_float2(ref[r], sum[r]);
    }
  window_codes<DT, D, RT, LY_THREADS>(p, gr.g, smem, q, row0, active, ks, wk, p.stat_tables, sp * p.stat_tables, p.stat_splits * p.stat_tables);
}

// ---------------------------------------------------------------------------------------------
// Scores, sign bits and counts.  Workgroup = (group, range of block keys).  Window rows and hyperplanes are A operands
// that stay in registers, keys the B operand: lane = key.  Waves 0-3 hold the window rows (RT tiles each) and pool the
// probabilities of a key in-lane over their rows; they do nothing else, and the exponentials of one pair of row tiles
// run beside the matrix work of the next.  Waves 4-7 hold the hyperplanes (PT tiles each): they take the sign bits,
// bring the keys into LDS, and finish the previous chunk (sums and sign bits meet in LDS, two buffers): the sum over
// the score waves, and per key and table one probe of the table's cells.  Every SIMD runs one wave of either kind.
// Both kinds have their instructions in a fixed order where a chunk is complete: a score wave four vector instructions and
// two exponentials beside each matrix instruction (exponents a step ahead of their exponentials, sums a step behind), a
// hashing wave two of the previous plane tile's signs.  A hashing wave first finishes the chunk before, served before the
// score wave of its SIMD, and then takes its products on equal terms: what is left at the barrier is then the score waves'
// (128k layer 227 -> 214-218 us, 64k 74.7 -> 68.5, 16k 23.6 -> 22.7, groups of eight 249 -> 240-245; with the hashing waves
// served first throughout and finishing last 227, never served first 251; ranges shorter than a chunk, where nothing is
// interleaved, the same within 1 %: layers in blocks of 72, 128 and 256 keys 37.0 -> 36.5, 32.9 -> 33.0, 39.3 -> 39.0).  Keys
// arrive by asynchronous loads (KeyRing); partials of the statistics are fetched eight at a time.  What the counting needs is
// computed from the thread's number chunk by chunk: kept in registers across the loop it went to scratch memory, whose loads
// wait for the keys on their way (groups of eight 267 us instead of 246, one chunk per workgroup 21.1 instead of 18.9).
// ---------------------------------------------------------------------------------------------
constexpr int LY_HALF = LY_WAVES / 2;  // waves of either kind

// COPIES: the hashing waves copy protected rows too
template <int DT, int D, int RT, int PT, bool COPIES>
__global__ __launch_bounds__(LY_THREADS) void layer_score_kernel(LayerParams p) {
  constexpr int ES = DT == DT_BF16 ? 2 : 4;
  constexpr int CH = D * ES / 16, NCH = CH / 2;
  using L = KeyRing<CH>;
  static_assert(L::KC == LY_KC, "a chunk of keys is a stage");
  constexpr int KC = LY_KC, TPC = KC / 32;
  constexpr int TP = RT > 1 ? 2 : 1;         // row tiles per step
  constexpr int NP = RT / TP;                // steps per key tile
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, rl = lane & 31, kg = lane >> 5;
  const int lin = xcd_major(blockIdx.x, gridDim.x);
  const LayerGroup gr = layer_group(p, lin / p.score_splits);
  const int k_lo = (lin % p.score_splits) * p.score_keys, k_hi = min(k_lo + p.score_keys, gr.s_t);
  if (k_lo >= k_hi) return;  // a short last block may leave ranges empty
  const int lim0 = gr.s_t - p.w;  // block key i is visible to window row j iff i <= lim0 + j
  const int n_rt = (p.m_rows + 31) >> 5, n_pt = (p.n_planes + 31) >> 5;
  const bool hash = wave >= LY_HALF;
  const int idx = wave & (LY_HALF - 1);
  // tiles of this wave: first, first + 4, ...; with fewer than three tiles several waves share one over different key
  // tiles (k0, k0 + kstep, ...)
  const int n_own = hash ? n_pt : n_rt;
  const int share = n_own >= 3 ? LY_HALF : n_own;
  const int kstep = LY_HALF / share, first = idx % share, k0 = idx / share;
  const bool active = first < n_own;
  const int n_sum = min(n_rt, LY_HALF);  // score waves whose sums make up a key's

  const int bits_pitch = (n_pt + 1) | 1;  // words per key in the sign-bit scratch: odd, and one past the last tile
  extern __shared__ uint4 smem[];
  uint32_t* sBits = reinterpret_cast<uint32_t*>(reinterpret_cast<char*>(smem) + 2 * L::STAGE);  // [2][KC][bits_pitch], behind two stages of keys
  float* sCol = reinterpret_cast<float*>(sBits + 2 * KC * bits_pitch);                      // [2][LY_HALF][KC]
  int* sLim = reinterpret_cast<int*>(sCol + 2 * LY_HALF * KC);                              // [LY_ROWS]
  float* sLse = reinterpret_cast<float*>(sLim + LY_ROWS);                                   // [LY_ROWS]
  uint32_t* sCells = reinterpret_cast<uint32_t*>(sLse + LY_ROWS);                             // [n_tables][cell_words]

  const uint32_t kstride = (uint32_t)p.k.stride_row;
  const srd_words ksrd =
      make_srd_words(p.k.base + (int64_t)gr.h * p.k.stride_head + (int64_t)gr.lo * p.k.stride_row, (uint32_t)gr.s_t * kstride);
  // LDS addresses of the lane's row in the first tile of a chunk: operand chunk pair i is at from[i % NA] + i / NA * (NA * 32)
  const uint32_t lds0 = lds_offset(smem);
  uint32_t from[L::NA];
  auto read_from = [&](int stage) {
#pragma unroll
    for (int i = 0; i < L::NA; ++i)
      from[i] = opaque(lds0 + stage * L::STAGE + rl / L::RPG * L::GROUP + rl % L::RPG * (CH * 16) + (((2 * i + kg) ^ (rl % L::RPG)) * 16));
  };
  auto key = [&](int tile, int i) { return lds_ld16(from[i % L::NA], tile * L::TILE + i / L::NA * (L::NA * 32)); };

  // the row's log-sum-exp (exp2 domain): merged from the partials of layer_stats_kernel and the caller's outside
  // keys, or the caller's complete one; and the cells
  auto rows_and_cells = [&]() {
    const int m = tid;
    float lse = 1.0e30f;  // padding rows: probability 0
    if (m < p.m_rows) {
      const float* outside = p.row_lse_blk ? p.row_lse_blk[gr.b] : p.row_lse;
      const float ext = outside ? outside[(size_t)gr.h * p.m_rows + m] * 1.4426950408889634f : 0.0f;
      if (p.lse_complete) {
        lse = ext;
      } else {
        float mm = NEG_BIG, ss = 0.0f;
        const float2* part = p.part + ((size_t)gr.g * p.m_rows + m) * p.n_parts;
        for (int i0 = 0; i0 < p.n_parts; i0 += 8) {  // eight loads in flight (one after another: a round trip each)
          float2 v[8];
#pragma unroll
          for (int u = 0; u < 8; ++u) v[u] = part[min(i0 + u, p.n_parts - 1)];
#pragma unroll
          for (int u = 0; u < 8; ++u)
            if (i0 + u < p.n_parts) lse_merge(mm, ss, v[u].x, v[u].y);
        }
        if (outside) lse_merge(mm, ss, ext, 1.0f);
        lse = lse_log2(mm, ss);
      }
    }
    sLse[m] = lse;
    const int mc = min(m, p.m_rows - 1);
    sLim[m] = lim0 + mc - div_w(mc, p.w_magic) * p.w;
    if (p.cells) {
      const int n_cw = p.n_tables * p.cell_words;
      const uint32_t* src = p.cells + (size_t)gr.g * n_cw;
      const int whole = (n_cw & 3) == 0 ? n_cw >> 8 : 0;  // KiB that go straight to LDS
      const srd_words csrd = make_srd_words(src, (uint32_t)n_cw * 4u);
      for (int kb = wave; kb < whole; kb += LY_WAVES) async_ld16(csrd, lane * 16, kb << 10, lds_offset(sCells) + (kb << 10));
      for (int i = (whole << 8) + tid; i < n_cw; i += LY_THREADS) sCells[i] = src[i];
      async_wait();
    }
  };
  // Operands of a wave's tiles.  Each kind of wave has its own, complete before its loop: what the compiler waits for at
  // their first use there would be waited for in every round.
  if (!hash) {
    uint4 a[RT][NCH];
#pragma unroll
    for (int t = 0; t < RT; ++t) {
      const char* ptr = layer_row(p, gr, min((first + LY_HALF * t) * 32 + rl, p.m_rows - 1));
#pragma unroll
      for (int i = 0; i < NCH; ++i) a[t][i] = ld16(ptr + (2 * i + kg) * 16);
    }
    rows_and_cells();
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
      for (int i = 0; i < NCH; ++i) landed(a[t][i]);
    __syncthreads();
    // logits of one step: row tiles t0, t0 + 1 against the 32 keys at LDS rows kt * 32 ..
    auto logits = [&](int kt, int t0, f32x16* acc) {
#pragma unroll
      for (int t = 0; t < TP; ++t)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[t][e] = 0.0f;
      uint32_t base[L::NA];  // kt is not a constant here
#pragma unroll
      for (int i = 0; i < L::NA; ++i) base[i] = from[i] + kt * L::TILE;
#pragma unroll
      for (int i = 0; i < NCH; ++i) {
        const uint4 kf = lds_ld16(base[i % L::NA], i / L::NA * (L::NA * 32));
#pragma unroll
        for (int t = 0; t < TP; ++t) Mma<DT>::run(acc[t], a[t0 + t][i], kf);
      }
    };
    // their probabilities, summed over the rows
    auto pooled = [&](const f32x16* acc, int t0) -> float {
      float c[TP];
#pragma unroll
      for (int t = 0; t < TP; ++t) {
        const int row = min((first + LY_HALF * (t0 + t)) * 32, LY_ROWS - 32);
        c[t] = 0.0f;
#pragma unroll
        for (int g4 = 0; g4 < 4; ++g4) {
          const float4 l4 = *reinterpret_cast<const float4*>(&sLse[row + acc_row(4 * g4, kg)]);
          const float ls[4] = {l4.x, l4.y, l4.z, l4.w};
#pragma unroll
          for (int u = 0; u < 4; ++u) c[t] += fast_exp2(fmaf(acc[t][4 * g4 + u], p.scale2, -ls[u]));
        }
      }
      return TP > 1 ? c[0] + c[TP - 1] : c[0];
    };
    auto pooled_masked = [&](const f32x16* acc, int t0, int kidx) -> float {
      float c = 0.0f;
#pragma unroll
      for (int t = 0; t < TP; ++t) {
        const int row = min((first + LY_HALF * (t0 + t)) * 32, LY_ROWS - 32);
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const float v = fast_exp2(fmaf(acc[t][e], p.scale2, -sLse[row + acc_row(e, kg)]));
          c += kidx <= sLim[row + acc_row(e, kg)] ? v : 0.0f;
        }
      }
      return c;
    };
    constexpr int PER = 16 / NCH;  // logits of a step per matrix instruction
    auto lse_of = [&](int t0, int g) {  // of four consecutive rows of the lane
      return *reinterpret_cast<const float4*>(&sLse[(first + LY_HALF * (t0 + g % TP)) * 32 + acc_row(4 * (g / TP), kg)]);
    };
    uint4 kf[NCH];
    float4 l[2] = {lse_of(0, 0), lse_of(0, 1)};  // those of the next logits
    int cur = 0;
    for (int kc0 = k_lo; kc0 < k_hi; kc0 += KC) {
      read_from(cur);
      float* col_dst = sCol + (size_t)(cur * LY_HALF + first) * KC;
      auto put = [&](int kt, float col) {
        col = half_pair_sum(col);
        const int l = fresh(lane);
        if (l < 32) col_dst[kt * 32 + l] = col;
      };
      if (kstep == 1 && kc0 + KC <= k_hi && kc0 + KC - 1 <= lim0) {  // workgroup-uniform: a complete chunk that every row sees
#pragma unroll
        for (int i = 0; i < NCH; ++i) kf[i] = key(0, i);
        f32x16 acc[2][TP];
        float c[TP];
#pragma unroll
        for (int t = 0; t < TP; ++t) c[t] = 0.0f;
#pragma unroll
        for (int s = 0; s <= TPC * NP; ++s) {
          // the products of step s beside the probabilities of step s - 1; what stands between two fences is issued
          // beside one matrix instruction
          const bool mul = s < TPC * NP, sum = s > 0, newk = mul && (s + 1) % NP == 0 && s + 1 < TPC * NP;
          f32x16* next = acc[s & 1];
          f32x16* done = acc[(s + 1) & 1];
          const int t0 = s % NP * TP, d0 = (s + NP - 1) % NP * TP;
          if (mul)
#pragma unroll
            for (int t = 0; t < TP; ++t)
#pragma unroll
              for (int e = 0; e < 16; ++e) next[t][e] = 0.0f;
          float x[PER], y[PER];
          auto exponents = [&](int j) {
#pragma unroll
            for (int k = 0; k < PER; ++k) {
              const int q = j * PER + k, g = q / 4;  // logits of four consecutive rows, tile by tile, and their log-sum-exps
              const float4 l4 = l[g & 1];
              const float ls = (q & 3) == 0 ? l4.x : (q & 3) == 1 ? l4.y : (q & 3) == 2 ? l4.z : l4.w;
              x[k] = fmaf(done[g % TP][4 * (g / TP) + (q & 3)], p.scale2, -ls);
              if ((q & 3) == 3) l[g & 1] = g + 2 < 4 * TP ? lse_of(d0, g + 2) : lse_of(t0, g + 2 - 4 * TP);
            }
          };
          auto sums = [&](int j) {
#pragma unroll
            for (int k = 0; k < PER; ++k) c[(j * PER + k) / 4 % TP] += y[k];
          };
          if (sum) exponents(0);
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int j = 0; j < NCH * TP; ++j) {
            const int i = j / TP, t = j % TP;
            if (mul) Mma<DT>::run(next[t], a[t0 + t][i], kf[i]);
            if (newk && t == TP - 1) kf[i] = key((s + 1) / NP, i);
            if (sum) {
              if (j > 0) sums(j - 1);
#pragma unroll
              for (int k = 0; k < PER; ++k) y[k] = fast_exp2(x[k]);
              if (j + 1 < NCH * TP) exponents(j + 1);
            }
            __builtin_amdgcn_sched_barrier(0);
          }
          if (sum) {
            sums(NCH * TP - 1);
            if (s % NP == 0) {
              put(s / NP - 1, TP > 1 ? c[0] + c[TP - 1] : c[0]);
#pragma unroll
              for (int t = 0; t < TP; ++t) c[t] = 0.0f;
            }
          }
        }
      } else if (active) {
#pragma unroll 1
        for (int kt = k0; kt < TPC; kt += kstep) {
          const int kbase = kc0 + kt * 32;
          if (kbase >= k_hi) break;  // wave-uniform
          float col = 0.0f;
#pragma unroll
          for (int t0 = 0; t0 < RT; t0 += TP) {
            f32x16 acc[TP];
            logits(kt, t0, acc);
            col += kbase + 31 <= lim0 ? pooled(acc, t0) : pooled_masked(acc, t0, kbase + rl);
          }
          put(kt, col);
        }
      }
      cur ^= 1;
      lds_barrier();
    }
    return;
  }

  // the hashing waves
  __builtin_amdgcn_s_setprio(1);
  // They bring the keys in: wave w of the four the w-th of every four groups of a stage; rows past the range's end repeat its
  // last one.
  const uint32_t ld_row = lane / CH, ld_col = ((lane % CH) ^ (ld_row % L::RPG)) * 16, ld_off = ld_row * kstride + ld_col;
  auto prefetch = [&](int kc0, int stage) {
    const int row = kc0 + idx * L::RPG;
    uint32_t dst = lds0 + stage * L::STAGE + idx * L::GROUP;
    constexpr int LOADS = KC / L::RPG / LY_HALF;
    if (kc0 + KC <= k_hi) {
      uint32_t src = (uint32_t)row * kstride;
#pragma unroll
      for (int u = 0; u < LOADS; ++u, src += LY_HALF * L::RPG * kstride, dst += LY_HALF * L::GROUP) async_ld16(ksrd, ld_off, src, dst);
    } else {
#pragma unroll 1
      for (int u = 0; u < LOADS; ++u, dst += LY_HALF * L::GROUP)
        async_ld16(ksrd, (uint32_t)min(row + u * LY_HALF * L::RPG + (int)ld_row, k_hi - 1) * kstride + ld_col, 0u, dst);
    }
  };
  prefetch(k_lo, 0);
  // One plane tile more than a multiple of the hashing waves: each of them holds it and takes it for one key tile of a chunk.  On
  // one wave it made that wave's SIMD do a quarter more matrix work than the others, and the barrier waits for it (64k layer,
  // 160 hyperplanes, 165.2 -> 162.5 us; 16k 57.4 -> 57.3).  Two or three tiles more are not shared out: the copies would cost
  // registers; nor is the thirteenth (four tiles a wave, where none are left).
  constexpr bool CAN_SPREAD = PT == 2 || PT == 3;
  const bool spread = CAN_SPREAD && n_pt == LY_HALF * (PT - 1) + 1;
  uint4 a[PT][NCH];
#pragma unroll
  for (int t = 0; t < PT; ++t) {
    const int tile = t == PT - 1 && spread ? n_pt - 1 : first + LY_HALF * t;
    const char* ptr = p.planes + (size_t)min(tile * 32 + plane_row(rl), p.n_planes - 1) * (D * ES);
#pragma unroll
    for (int i = 0; i < NCH; ++i) a[t][i] = ld16(ptr + (2 * i + kg) * 16);
  }
  rows_and_cells();
#pragma unroll
  for (int t = 0; t < PT; ++t)
#pragma unroll
    for (int i = 0; i < NCH; ++i) landed(a[t][i]);
  async_wait();
  __syncthreads();
  const uint32_t code_mask = (1u << p.n_bits) - 1u;
  const uint32_t cell_max = p.cell_log == 2 ? 255u : 15u;  // full cells of 8 and 4 bits (cell_log 2, 3; those of 16 bits hold every count)
  // sums over the score waves and collision counts of the chunk whose first key is kc0: two lanes per key
  auto finish = [&](int buf, int kc0) {
    const int at_tid = fresh(tid), key = (at_tid - LY_HALF * 64) >> 1, sub = at_tid & 1;
    const int kidx = kc0 + key;
    const uint32_t* bits = sBits + (buf * KC + key) * bits_pitch;
    const size_t at = (size_t)gr.g * p.s_stride + kidx;
    if (sub == 0 && kidx < k_hi) {
      const float* col = sCol + (size_t)buf * LY_HALF * KC + key;
      float v = col[0];
      for (int w = 1; w < n_sum; ++w) v += col[w * KC];
      p.score[at] = v;
    }
    auto code_of = [&](int t) {
      const int bitpos = t * p.n_bits, w0 = bitpos >> 5;
      return __builtin_amdgcn_alignbit(bits[w0 + 1], bits[w0], bitpos & 31) & code_mask;
    };
    if (p.cells) {
      uint32_t n = 0u, fullest = 0u;
      auto nibble_of = [&](int t, uint32_t code) {
        return __builtin_amdgcn_ubfe(sCells[t * p.cell_words + (code >> 3)], (code & 7u) << 2, 4u);
      };
      // cells are read at their own width: the barrier waits for the counting
      if (p.cell_log == 1) {
#pragma unroll 8
        for (int t = sub; t < p.n_tables; t += 2)
          n += reinterpret_cast<const uint16_t*>(sCells + t * p.cell_words)[code_of(t)];
      } else if (p.cell_log == 2) {
#pragma unroll 8
        for (int t = sub; t < p.n_tables; t += 2) {
          const uint32_t c = reinterpret_cast<const uint8_t*>(sCells + t * p.cell_words)[code_of(t)];
          n += c;
          fullest = max(fullest, c);
        }
      } else {
#pragma unroll 8
        for (int t = sub; t < p.n_tables; t += 2) {
          const uint32_t c = nibble_of(t, code_of(t));
          n += c;
          fullest = max(fullest, c);
        }
      }
      if (p.cell_log > 1 && __any(fullest == cell_max)) {  // some key met a heavy bin: its count is in the table's list
        for (int t = sub; t < p.n_tables; t += 2) {
          const uint32_t code = code_of(t);
          const uint32_t c = p.cell_log == 2 ? reinterpret_cast<const uint8_t*>(sCells + t * p.cell_words)[code] : nibble_of(t, code);
          if (c != cell_max) continue;
          const uint32_t* list = p.heavy + ((size_t)gr.g * p.n_tables + t) * LY_HEAVY;
          const int len = (int)list[0];
          for (int i = 1; i <= len; ++i)
            if (list[i] >> 16 == code) n += (list[i] & 0xffffu) - cell_max;
        }
      }
      n += lane_xor1(n);
      if (sub == 0 && kidx < k_hi) p.cnt[at] = (int)n;
    } else if (kidx < k_hi) {
      if (code_octets(p.n_tables)) {
        const int n_oct = p.n_tables >> 3;
        for (int o = sub; o < n_oct; o += 2) {
          uint32_t two[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) two[u] = code_of(8 * o + 2 * u) | code_of(8 * o + 2 * u + 1) << 16;
          *reinterpret_cast<uint4*>(p.sig_k + (((size_t)gr.g * n_oct + o) * p.s_stride + kidx) * 8) = make_uint4(two[0], two[1], two[2], two[3]);
        }
      } else {
        uint16_t* dst = p.sig_k + at * p.n_tables;
        for (int t = sub; t < p.n_tables; t += 2) dst[t] = (uint16_t)code_of(t);
      }
      if (sub == 1) p.cnt[at] = 0;  // count_kernel accumulates with atomics
    }
  };
  // Rows that are kept whatever the scores (the block's first n_anchor and last n_local) go to the cache from here: this
  // kernel leaves the memory idle, and the selection behind it, which is bound by it, has so much less to copy (a quarter to
  // a half of the kept rows at divisors of 8 and 4).  A piece is 16 bytes of a key and of its value; each range takes a share
  // of them, its threads two a chunk, loaded in one chunk and stored in the next; what is left then (divisors below 4 and
  // larger budgets) follows behind the last chunk.  Offsets are 32-bit ones into descriptors (64-bit addresses took 0.5 us a
  // chunk), past whose end nothing is loaded or stored.
  constexpr int PIECES = 2, STEP = LY_HALF * 64 / CH;  // rows from one of a thread's pieces to its next
  const bool last_blk = gr.b == p.n_blocks - 1;
  const int n_front = last_blk ? p.last_anchor : p.n_anchor, n_prot = n_front + (last_blk ? p.last_local : p.n_local);
  const int n_kept = last_blk ? p.last_kept : p.n_kept, rows_of = last_blk ? p.last_copies : p.copies;
  int row0 = lin % p.score_splits * rows_of;  // protected rows from here on are still to be stored
  const int row_end = COPIES ? min(row0 + rows_of, n_prot) : 0;
  uint4 k_piece[PIECES], v_piece[PIECES];
  auto each_piece = [&](auto f) {  // (which, row among the protected ones, byte in the row)
    const int t = fresh(tid) - LY_HALF * 64;
#pragma unroll
    for (int u = 0; u < PIECES; ++u) f(u, row0 + t / CH + u * STEP, (uint32_t)(t % CH * 16));
  };
  auto fetch_pieces = [&]() {
    const int h = fresh_scalar(gr.h);
    const __amdgpu_buffer_rsrc_t ks = make_srd(p.k.base + (int64_t)h * p.k.stride_head + (int64_t)gr.lo * p.k.stride_row, (uint32_t)gr.s_t * kstride);
    const uint32_t vstride = (uint32_t)p.v.stride_row;
    const __amdgpu_buffer_rsrc_t vs = make_srd(p.v.base + (int64_t)h * p.v.stride_head + (int64_t)gr.lo * p.v.stride_row, (uint32_t)gr.s_t * vstride);
    each_piece([&](int u, int j, uint32_t c) {
      const uint32_t token = j < n_front ? j : gr.s_t - n_prot + j;  // past the last one: past the block
      k_piece[u] = buf_ld16(ks, token * kstride + c);
      v_piece[u] = buf_ld16(vs, token * vstride + c);
    });
  };
  auto store_pieces = [&]() {
    const int64_t at = (int64_t)fresh_scalar(gr.h) * p.cache_stride_head + (int64_t)gr.b * p.n_kept * (CH * 16);
    const uint32_t bytes = (uint32_t)n_kept * (CH * 16);
    const __amdgpu_buffer_rsrc_t ks = make_srd(p.k_cache + at, bytes), vs = make_srd(p.v_cache + at, bytes);
    each_piece([&](int u, int j, uint32_t c) {
      const uint32_t row = j >= row_end ? 0x00ffffffu : j < n_front ? j : n_kept - n_prot + j;
      buf_st16_stream(ks, row * (CH * 16) + c, k_piece[u]);
      buf_st16_stream(vs, row * (CH * 16) + c, v_piece[u]);
    });
    row0 += PIECES * STEP;
  };
  int cur = 0;
  for (int kc0 = k_lo; kc0 < k_hi; kc0 += KC) {
    const bool more = kc0 + KC < k_hi;
    __builtin_amdgcn_s_setprio(1);
    if (COPIES && kc0 > k_lo && row0 < row_end) store_pieces();  // before the keys' loads: what they wait for has landed
    if (more) prefetch(kc0 + KC, cur ^ 1);
    read_from(cur);
    if (kc0 > k_lo) finish(cur ^ 1, kc0 - KC);
    if (COPIES && row0 < row_end) fetch_pieces();
    __builtin_amdgcn_s_setprio(0);
    if (active && kstep == 1 && kc0 + KC <= k_hi) {  // a complete chunk
      // The products of a (key tile, plane tile) beside the sign bits of the one before.
      auto steps = [&](auto tiles, auto more_tiles) {
        constexpr int N = decltype(tiles)::value;  // plane tiles of this wave
        constexpr int M = TPC * N + decltype(more_tiles)::value;  // products; the last one of the tile that all waves hold
        constexpr int PER = 16 / NCH;
        static_assert(TPC == LY_HALF, "a key tile of the chunk for each hashing wave");
        uint32_t* bits = sBits + (cur * KC + rl) * bits_pitch + first;
        uint4 kf[NCH];
        f32x16 acc[2];
#pragma unroll
        for (int i = 0; i < NCH; ++i) kf[i] = key(0, i);
#pragma unroll
        for (int s = 0; s <= M; ++s) {
          const bool mul = s < M, newk = s < TPC * N && s % N == N - 1 && (s / N + 1 < TPC || M > TPC * N);
          uint32_t neg = 0u;
          if (mul)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[s & 1][e] = 0.0f;
#pragma unroll
          for (int i = 0; i < NCH; ++i) {
            if (mul) Mma<DT>::run(acc[s & 1], a[s < TPC * N ? s % N : PT - 1][i], kf[i]);
            if (newk) kf[i] = s / N + 1 < TPC ? key(s / N + 1, i) : lds_ld16(from[i % L::NA] + first * L::TILE, i / L::NA * (L::NA * 32));
            if (s > 0)
#pragma unroll
              for (int e = i * PER; e < (i + 1) * PER; ++e) neg = __builtin_amdgcn_alignbit(neg, __float_as_uint(acc[(s + 1) & 1][15 - e]), 31);
            __builtin_amdgcn_sched_barrier(0);
          }
          if (s > 0) {
            // 16 consecutive planes per lane (see plane_row): their sign bits have been shifted into one word
            const uint32_t pos = ~neg & 0xffffu;
            const uint32_t mask = pos | (half_other(pos, kg) << 16);
            if (kg == 0) {
              if (s <= TPC * N) bits[(s - 1) / N * 32 * bits_pitch + LY_HALF * ((s - 1) % N)] = mask;
              else bits[first * 32 * bits_pitch + n_pt - 1 - first] = mask;
            }
          }
        }
      };
      constexpr std::integral_constant<int, PT == 1 ? 1 : PT - 1> fewer;
      constexpr std::integral_constant<int, 0> none;
      if (spread) steps(fewer, std::integral_constant<int, CAN_SPREAD>{});
      else if (first + LY_HALF * (PT - 1) < n_pt) steps(std::integral_constant<int, PT>{}, none);
      else steps(fewer, none);
    } else if (active) {
#pragma unroll 1
      for (int vt = k0; vt < TPC; vt += kstep) {
        if (kc0 + vt * 32 >= k_hi) break;
        auto signs = [&](const f32x16& acc, int t) {
          // 16 consecutive planes per lane (see plane_row): their sign bits shift into one word
          uint32_t neg = 0u;
#pragma unroll
          for (int e = 15; e >= 0; --e) neg = __builtin_amdgcn_alignbit(neg, __float_as_uint(acc[e]), 31);
          const uint32_t pos = ~neg & 0xffffu;
          const uint32_t mask = pos | (half_other(pos, kg) << 16);
          const int tile = t == PT - 1 && spread ? n_pt - 1 : first + LY_HALF * t;  // (all four write the same)
          if (kg == 0 && tile < n_pt) sBits[(cur * KC + vt * 32 + rl) * bits_pitch + tile] = mask;
        };
        constexpr int HT = PT == 4 ? 2 : PT;  // tiles at a time (registers)
#pragma unroll
        for (int t0 = 0; t0 < PT; t0 += HT) {
          f32x16 acc[HT];
#pragma unroll
          for (int t = 0; t < HT; ++t)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[t][e] = 0.0f;
#pragma unroll
          for (int i = 0; i < NCH; ++i) {
            const uint4 kf = lds_ld16(from[i % L::NA] + vt * L::TILE, i / L::NA * (L::NA * 32));
#pragma unroll
            for (int t = 0; t < HT; ++t) Mma<DT>::run(acc[t], a[t0 + t][i], kf);
          }
#pragma unroll
          for (int t = 0; t < HT; ++t) signs(acc[t], t0 + t);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
    if (more) async_wait();
    cur ^= 1;
    lds_barrier();
  }
  finish(cur ^ 1, k_lo + (k_hi - k_lo - 1) / KC * KC);
  while (COPIES && row0 < row_end) {
    store_pieces();
    if (row0 < row_end) fetch_pieces();
  }
}

// ---- host side ----
bool layer_supports(int dtype, int head_dim, int m_rows) {
  return head_dim * (dtype == DT_BF16 ? 2 : 4) <= 256 && m_rows <= LY_ROWS;
}

static size_t score_lds(int head_dim, int es, int n_planes, int cell_total_words) {
  const int bits_pitch = ((n_planes + 31) / 32 + 1) | 1;
  const size_t stage = head_dim * es <= 128 ? KeyRing<8>::STAGE : KeyRing<16>::STAGE;
  return 2 * stage + (size_t)2 * LY_KC * bits_pitch * 4 +
         (size_t)2 * LY_HALF * LY_KC * 4 + (size_t)LY_ROWS * 8 + (size_t)cell_total_words * 4 + 16;
}

// Whether the score kernel copies the blocks' protected rows (us a layer: the selection copies them, this kernel does).
//  - It has at least three chunks per workgroup to load and store in (64 groups of four ranges of one chunk 34.3, 35.3; of two
//    46.0, 46.2; of three 51.1, 48.9), and at least a fifth of the kept rows are protected (16 blocks of 4096 at a divisor of
//    8 250.7, 244.8; 32 blocks of 2048 at 10 167.1, 166.6, at 12 166.6, 167.0, at 16 166.4, 168.1).
//  - Plane tiles leave registers (four a wave: 60 bytes in scratch memory, groups of eight 577, 600).
//  - Its workgroups fill most of the chip.  Where they do not, neither do the selection's, which are no slower for the rows
//    (groups of sixteen ranges of 512 keys: two groups 55.1, 56.2, four 55.0, 56.3, eight 56.4, 57.5; ten 59.8, 60.2, and at
//    twice the budget 76.9, 63.6; twelve 61.1, 60.1).
//  - A range has enough of them for what each workgroup pays: where a block is one range 48 (ranges of 384 keys with 40 of them
//    52.2, 52.4, with 93 52.1, 50.8; of 512 with 62 60.2, 59.1), else 16 KiB of each tensor (four ranges of 512 keys, rows of 256
//    bytes: 57 of them 61.0, 61.8, with 384 hyperplanes 69.9, 72.0; 60 61.5, 62.3; 76 60.2, 59.7; 114 60.9, 59.3, of 128 bytes
//    43.0, 44.1).
// Rows of 128 bytes and fp32 likewise (128k layer of dimension 64 at a divisor of 4 349.5, 334.5, fp32 layer of 32k 224.4,
// 214.2).  There is no line above which it copies too many: at a divisor of 2 and twice the budget, where half of them are left
// to the loop behind the last chunk, 128k layer 655, 612, 64k 219, 205, 16k 70.7, 69.0.
static bool copies_protected(const LayerParams& p, int row_bytes, int n_cu, int rows) {
  const int64_t n_wg = (int64_t)p.n_blocks * p.n_kv_heads * p.score_splits;
  return p.score_keys >= 3 * LY_KC && 5 * (p.n_anchor + p.n_local) >= p.n_kept && p.n_planes <= 3 * 32 * LY_HALF &&
         8 * n_wg >= 5 * n_cu && (p.score_splits == 1 ? rows >= 48 : rows * row_bytes >= 16 * 1024);
}

void layer_plan_copies(int row_bytes, int n_cu, LayerParams* p) {
  auto rows = [&](int s_t, int n_prot) {  // per range with keys
    const int n_rng = (s_t + p->score_keys - 1) / p->score_keys;
    return (n_prot + n_rng - 1) / n_rng;
  };
  const int each = rows(p->s_block, p->n_anchor + p->n_local);
  const bool copies = copies_protected(*p, row_bytes, n_cu, each) && (int64_t)p->s_block * p->v.stride_row < (int64_t(1) << 31);  // 32-bit offsets
  p->copies = copies ? each : 0;
  p->last_copies = copies ? rows(p->n_tok - (p->n_blocks - 1) * p->s_block, p->last_anchor + p->last_local) : 0;
}

// Key ranges per group: workgroups come in rounds of n_cu (one per compute unit); a workgroup costs its keys plus
// `ovh` (its loads of rows and hyperplanes, in units of keys).
static int best_splits(int n_groups, int keys, int n_cu, int ovh, int* per) {
  int best = 1;
  long best_cost = -1;
  for (int s = 1; s <= 16; ++s) {
    const int kps = (keys + s - 1) / s, k32 = (kps + 31) / 32 * 32;
    const long cost = (long)((n_groups * s + n_cu - 1) / n_cu) * (k32 + ovh);
    if (best_cost < 0 || cost < best_cost) {
      best_cost = cost;
      best = s;
      *per = k32;
    }
  }
  return best;
}

void layer_plan(int dtype, int head_dim, int n_cu, LayerParams* p, LayerPlan* plan) {
  const int es = dtype == DT_BF16 ? 2 : 4;
  const int n_groups = p->n_blocks * p->n_kv_heads;
  const int n_rt = (p->m_rows + 31) / 32;
  plan->rt = n_rt > 4 ? 2 : 1;
  const int need = (n_rt + plan->rt - 1) / plan->rt;
  p->wr_log = 0;
  while ((1 << p->wr_log) < need) ++p->wr_log;
  p->stat_splits = best_splits(n_groups, p->s_block + p->n_ctx, n_cu, 160, &p->stat_keys);
  p->score_splits = best_splits(n_groups, p->s_block, n_cu, 128, &p->score_keys);
  p->n_parts = p->stat_splits * (LY_WAVES >> p->wr_log);
  p->s_stride = (p->s_block + 3) & ~3;
  // tables per pass of the code kernel: histograms within 68 KiB, at most 256 hyperplanes
  const int words = p->n_bits >= 5 ? 1 << (p->n_bits - 5) : 1;
  int cw = 0;
  plan->use_cells = 0;
  for (p->cell_log = 1; p->n_bits <= 12 && p->cell_log <= 3 && !plan->use_cells; ++p->cell_log) {
    cw = max(1, (1 << p->n_bits) >> p->cell_log);
    plan->use_cells = (size_t)cw * p->n_tables * 4 <= 64 * 1024 && score_lds(head_dim, es, p->n_planes, cw * p->n_tables) <= 160 * 1024;
    if (plan->use_cells) break;
  }
  p->cell_words = plan->use_cells ? cw : 0;
  int nt = LY_CODE_PLANES / p->n_bits;
  if (plan->use_cells) nt = min(nt, 1024 / words);
  p->code_tables = max(1, min(nt, p->n_tables));
  // groups that leave compute units idle share their tables out: smaller sets, one or more workgroups each (a 16k layer of
  // 64 groups: 10.2 -> 6.4 us)
  const int share = min(max(1, n_cu / n_groups), p->n_tables);
  p->code_tables = min(p->code_tables, (p->n_tables + share - 1) / share);
  plan->code_split = min(share, (p->n_tables + p->code_tables - 1) / p->code_tables);
  auto codes_lds = [&](int tables) {
    return (size_t)code_plane_rows(tables, p->n_bits) * (head_dim * es / 16 + 1) * 16 + (plan->use_cells ? (size_t)(tables * (words * 17 + 1) + 4) * 4 : 0);
  };
  plan->codes_lds = codes_lds(p->code_tables);
  // The statistics kernel takes the codes along, a group's tables shared out over its key ranges.  Where they need more than
  // one set, sets that fill whole tiles of hyperplanes (32 tables of 12 bits: eight at a time 177.5 us, eleven 179.1).
  const int tables_of = (p->n_tables + p->stat_splits - 1) / p->stat_splits;
  p->stat_tables = min(LY_CODE_PLANES / p->n_bits, tables_of);
  while (p->stat_tables > 1 && codes_lds(p->stat_tables) > 160 * 1024) --p->stat_tables;
  if (p->stat_tables < tables_of) {
    int whole = 1;
    while (whole * p->n_bits & 31) ++whole;
    if (whole <= p->stat_tables) p->stat_tables -= p->stat_tables % whole;
  }
  plan->stats_lds = max(row_stats_lds(head_dim * es), codes_lds(p->stat_tables));
  plan->score_lds = score_lds(head_dim, es, p->n_planes, plan->use_cells ? cw * p->n_tables : 0);
  // workspace
  auto up = [](size_t x) { return (x + 255) & ~(size_t)255; };
  const size_t g = n_groups;
  size_t off = 0;
  plan->off_part = off;   off += up(g * p->m_rows * p->n_parts * sizeof(float2));
  plan->off_score = off;  off += up(g * p->s_stride * sizeof(float));
  plan->off_cnt = off;    off += up(g * p->s_stride * sizeof(int32_t));
  plan->off_cells = off;    off += plan->use_cells ? up(g * p->n_tables * cw * sizeof(uint32_t)) : 0;
  plan->off_heavy = off;  off += plan->use_cells ? up(g * p->n_tables * LY_HEAVY * sizeof(uint32_t)) : 0;
  plan->off_sig_k = off;  off += plan->use_cells ? 0 : up(g * p->s_stride * p->n_tables * sizeof(uint16_t));
  plan->off_sig_q = off;  off += plan->use_cells ? 0 : up(g * p->m_rows * p->n_tables * sizeof(uint16_t));
  plan->bytes = off + 256;
}

template <int DT, int D>
static hipError_t launch_codes_t(const LayerParams& p, const LayerPlan& plan, hipStream_t st) {
  hipLaunchKernelGGL((layer_codes_kernel<DT, D>), dim3(p.n_blocks * p.n_kv_heads, plan.code_split), dim3(LY_CODE_THREADS), plan.codes_lds, st, p);
  return hipGetLastError();
}
template <int DT, int D>
static hipError_t launch_stats_t(const LayerParams& p, const LayerPlan& plan, hipStream_t st) {
  const dim3 grid(p.n_blocks * p.n_kv_heads * p.stat_splits);
  const bool lng = row_stats_long(DT, D * (DT == DT_BF16 ? 2 : 4), plan.rt, p.stat_keys);
  if (plan.rt == 2 && lng) hipLaunchKernelGGL((layer_stats_kernel<DT, D, 2, DT == DT_BF16>), grid, dim3(LY_THREADS), plan.stats_lds, st, p);
  else if (plan.rt == 2) hipLaunchKernelGGL((layer_stats_kernel<DT, D, 2, false>), grid, dim3(LY_THREADS), plan.stats_lds, st, p);
  else hipLaunchKernelGGL((layer_stats_kernel<DT, D, 1, false>), grid, dim3(LY_THREADS), plan.stats_lds, st, p);
  return hipGetLastError();
}
template <int DT, int D, int RT>
static hipError_t launch_score_rt(const LayerParams& p, const LayerPlan& plan, hipStream_t st) {
  const dim3 grid(p.n_blocks * p.n_kv_heads * p.score_splits), blk(LY_THREADS);
  const int pt = (p.n_planes + 32 * LY_HALF - 1) / (32 * LY_HALF);
  const bool copies = p.copies || p.last_copies;
  if (pt == 1 && copies) hipLaunchKernelGGL((layer_score_kernel<DT, D, RT, 1, true>), grid, blk, plan.score_lds, st, p);
  else if (pt == 1) hipLaunchKernelGGL((layer_score_kernel<DT, D, RT, 1, false>), grid, blk, plan.score_lds, st, p);
  else if (pt == 2 && copies) hipLaunchKernelGGL((layer_score_kernel<DT, D, RT, 2, true>), grid, blk, plan.score_lds, st, p);
  else if (pt == 2) hipLaunchKernelGGL((layer_score_kernel<DT, D, RT, 2, false>), grid, blk, plan.score_lds, st, p);
  else if (pt == 3 && copies) hipLaunchKernelGGL((layer_score_kernel<DT, D, RT, 3, true>), grid, blk, plan.score_lds, st, p);
  else if (pt == 3) hipLaunchKernelGGL((layer_score_kernel<DT, D, RT, 3, false>), grid, blk, plan.score_lds, st, p);
  else hipLaunchKernelGGL((layer_score_kernel<DT, D, RT, 4, false>), grid, blk, plan.score_lds, st, p);
  return hipGetLastError();
}
template <int DT, int D>
static hipError_t launch_score_t(const LayerParams& p, const LayerPlan& plan, hipStream_t st) {
  const int n_rt = (p.m_rows + 31) / 32;
  if (n_rt <= LY_HALF) return launch_score_rt<DT, D, 1>(p, plan, st);
  if (n_rt <= 2 * LY_HALF) return launch_score_rt<DT, D, 2>(p, plan, st);
  return launch_score_rt<DT, D, 4>(p, plan, st);
}

#define LY_DISPATCH(fn)                                                              \
  if (dtype == DT_BF16 && head_dim == 128) return fn<DT_BF16, 128>(p, plan, st);     \
  if (dtype == DT_BF16 && head_dim == 64) return fn<DT_BF16, 64>(p, plan, st);       \
  if (dtype == DT_F32 && head_dim == 64) return fn<DT_F32, 64>(p, plan, st);         \
  return hipErrorInvalidValue

hipError_t launch_layer_codes(int dtype, int head_dim, const LayerParams& p, const LayerPlan& plan, hipStream_t st) { LY_DISPATCH(launch_codes_t); }
hipError_t launch_layer_stats(int dtype, int head_dim, const LayerParams& p, const LayerPlan& plan, hipStream_t st) { LY_DISPATCH(launch_stats_t); }
hipError_t launch_layer_score(int dtype, int head_dim, const LayerParams& p, const LayerPlan& plan, hipStream_t st) { LY_DISPATCH(launch_score_t); }

static hipError_t allow_lds(const void* kernel) { return hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024); }
template <int DT, int D, int RT>
static hipError_t score_attrs() {
  const void* fns[] = {reinterpret_cast<const void*>(&layer_score_kernel<DT, D, RT, 1, false>), reinterpret_cast<const void*>(&layer_score_kernel<DT, D, RT, 1, true>),
                       reinterpret_cast<const void*>(&layer_score_kernel<DT, D, RT, 2, false>), reinterpret_cast<const void*>(&layer_score_kernel<DT, D, RT, 2, true>),
                       reinterpret_cast<const void*>(&layer_score_kernel<DT, D, RT, 3, false>), reinterpret_cast<const void*>(&layer_score_kernel<DT, D, RT, 3, true>),
                       reinterpret_cast<const void*>(&layer_score_kernel<DT, D, RT, 4, false>)};
  for (const void* f : fns) {
    const hipError_t e = allow_lds(f);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}
template <int DT, int D>
static hipError_t layer_attrs() {
  hipError_t e = allow_lds(reinterpret_cast<const void*>(&layer_codes_kernel<DT, D>));
  if (e == hipSuccess) e = allow_lds(reinterpret_cast<const void*>(&layer_stats_kernel<DT, D, 1, false>));
  if (e == hipSuccess) e = allow_lds(reinterpret_cast<const void*>(&layer_stats_kernel<DT, D, 2, false>));
  if (e == hipSuccess) e = allow_lds(reinterpret_cast<const void*>(&layer_stats_kernel<DT, D, 2, DT == DT_BF16>));
  if (e == hipSuccess) e = score_attrs<DT, D, 1>();
  if (e == hipSuccess) e = score_attrs<DT, D, 2>();
  if (e == hipSuccess) e = score_attrs<DT, D, 4>();
  return e;
}
hipError_t init_layer_attributes(int dtype, int head_dim) {
  if (dtype == DT_BF16) return head_dim == 128 ? layer_attrs<DT_BF16, 128>() : layer_attrs<DT_BF16, 64>();
  return head_dim == 64 ? layer_attrs<DT_F32, 64>() : hipSuccess;  // fp32 with rows of 512 bytes: layer_supports
}

}  // namespace lkv

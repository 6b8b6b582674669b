// Attention kernels for gfx950: over the compacted cache (Sec. 3 first paragraph: the kept tokens are what
// later tokens attend to; every cached row is visible, the cache holds earlier blocks only) and, behind the
// cache rows, over the current block's own keys under the causal mask (the block's prefill attention, whose
// log-sum-exp of the window rows is the complete statistic of Sec. 3.3 "Precision").
//
//   attend_decode_kernel   at most eight query rows per KV head over the cache (decoding): laserkv_decode.hip
//   attend_kernel          up to four row tiles otherwise (128 query rows per KV head).  Workgroup = (key split, KV head);
//                          the waves share row tiles over different key tiles.  The split's keys and
//                          values pass through LDS in chunks; each wave keeps 32 query rows in registers and an
//                          online-softmax state (reference, sum, unnormalised output) per row; the waves'
//                          states meet in LDS and leave one partial per split                          [MFMA]
//   attend_rows_kernel     more than four row tiles (window rows, whole blocks): two waves per pair of row tiles that
//                          together see the same number of keys, keys and values straight into two LDS stages; writes
//                          the result itself when a workgroup sees all keys of its rows                      [MFMA]
//   attend_combine_kernel  merges the partials of a row through their references and writes the output and
//                          the natural-log normaliser, the number laserkv_set_row_lse takes
//   attend_lse_kernel (+ attend_lse_combine_kernel)  the normaliser alone, for callers that want nothing else
#include "laserkv_device.h"
#include "laserkv_kernels.h"
#include "laserkv_rowstats.h"

namespace lkv {

constexpr int ATT_WAVES = 8;
constexpr int ATT_THREADS = ATT_WAVES * 64;
constexpr int ATT_ROWS = 256;      // query rows per workgroup: up to 8 row tiles
constexpr int ATT_MAX_SPLITS = 64;

// Keys per LDS chunk of attend_kernel (as many as its prefetch registers hold).
template <int DT>
__host__ __device__ constexpr int att_chunk_keys() { return DT == DT_BF16 ? 256 : 128; }

// Transposes, inside groups of 8 consecutive lanes, the 8 x 8 matrix of 16-bit elements whose row i is lane
// i's 16 bytes: afterwards lane i holds column i, element e of it being what lane e held at position i.
// Three exchange steps, each swapping one bit of the lane index with one bit of the element index; lane
// exchanges are DPP moves and every step is a select (no branches, no LDS traffic).
__device__ __forceinline__ uint4 transpose_8x8_b16(const uint4& v, int lane) {
  uint32_t x[4] = {v.x, v.y, v.z, v.w};
  const bool i0 = lane & 1, i1 = lane & 2, i2 = lane & 4;
  // lane bit 0 <-> half of the word: an even lane keeps its low half and takes the partner's low half as its
  // high half; an odd lane takes the partner's high half as its low half and keeps its high half
  const uint32_t sel = i0 ? 0x03020706u : 0x05040100u;  // byte picks from {partner (bytes 4-7), own (bytes 0-3)}
#pragma unroll
  for (int w = 0; w < 4; ++w) x[w] = __builtin_amdgcn_perm(lane_xor1(x[w]), x[w], sel);
#pragma unroll
  for (int a = 0; a < 4; a += 2) {  // lane bit 1 <-> word bit 0
    const uint32_t recv = lane_xor2(i1 ? x[a] : x[a + 1]);
    x[a] = i1 ? recv : x[a];
    x[a + 1] = i1 ? x[a + 1] : recv;
  }
#pragma unroll
  for (int a = 0; a < 2; ++a) {  // lane bit 2 <-> word bit 1
    const uint32_t recv = lane_xor4(i2 ? x[a] : x[a + 2], i2);
    x[a] = i2 ? recv : x[a];
    x[a + 2] = i2 ? x[a + 2] : recv;
  }
  return make_uint4(x[0], x[1], x[2], x[3]);
}

// The same for 4 x 4 matrices of 32-bit elements inside groups of 4 consecutive lanes.
__device__ __forceinline__ uint4 transpose_4x4_b32(const uint4& v, int lane) {
  uint32_t x[4] = {v.x, v.y, v.z, v.w};
  const bool i0 = lane & 1, i1 = lane & 2;
#pragma unroll
  for (int a = 0; a < 4; a += 2) {
    const uint32_t recv = lane_xor1(i0 ? x[a] : x[a + 1]);
    x[a] = i0 ? recv : x[a];
    x[a + 1] = i0 ? x[a + 1] : recv;
  }
#pragma unroll
  for (int a = 0; a < 2; ++a) {
    const uint32_t recv = lane_xor2(i1 ? x[a] : x[a + 2]);
    x[a] = i1 ? recv : x[a];
    x[a + 2] = i1 ? x[a + 2] : recv;
  }
  return make_uint4(x[0], x[1], x[2], x[3]);
}

// Writes one transposed group (the group's EPC consecutive keys at one head-dimension index) into that index's
// row of V^T.  fp32: keys in order.  bf16: the P operand of O^T += V^T P^T holds, per lane half kg and 16-key
// block, keys 4kg + (0..3) and 8 + 4kg + (0..3) (the accumulator layout of S^T); the row stores every 16-key
// block in that order, [0-3, 8-11 | 4-7, 12-15], so that a lane's eight keys are one 16-byte read.
template <int DT>
__device__ __forceinline__ void store_vt(uint4* row, int group, const uint4& t) {
  if (DT == DT_BF16) {
    uint2* r2 = reinterpret_cast<uint2*>(row) + 4 * (group >> 1) + (group & 1);
    r2[0] = make_uint2(t.x, t.y);
    r2[2] = make_uint2(t.z, t.w);
  } else {
    row[group] = t;
  }
}

// ds_read_b64_tr_b16: four 16-bit values per lane, transposed within groups of 16 lanes (see its use)
typedef short s16x4_lds __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint2 ds_read_tr16(uint32_t at) {
  const s16x4_lds v = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4_lds*)(uintptr_t)at);
  return __builtin_bit_cast(uint2, v);
}

__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  bf16x2 t = {(__bf16)lo, (__bf16)hi};  // round to nearest even
  return __builtin_bit_cast(uint32_t, t);
}

// One pass over the split's keys for launches with few query rows (the waves of a workgroup share row tiles
// over different key tiles): its share of the cache rows, then its share of the block's own keys (none
// for attention over the cache alone).  S^T = K Q^T puts a query row in a lane (column rl of the tile; the two
// halves kg of the wave hold the same rows over different keys), so the softmax state is lane-private, and
// the 16 accumulator registers are already the B operand of O^T += V^T P^T: register r of half kg is key
// acc_row(r, kg), so a group of 8 (bf16) or 4 (f32) registers is one 16-byte operand chunk whose keys the A
// operand matches by reading V^T at the same key offsets.  V is transposed in registers on its way into LDS.
// Block key i is visible to query j iff i <= diag + j: chunks past the last row of the workgroup are never
// loaded, tiles past the last row of the wave are skipped, tiles that cross a row's limit take a masked path.
template <int DT, int D, int KC>
__global__ __launch_bounds__(ATT_THREADS) void attend_kernel(AttendParams p) {
  constexpr int ES = DT == DT_BF16 ? 2 : 4;
  constexpr int CH = D * ES / 16;             // 16-byte chunks per row
  constexpr int NCH = CH / 2;
  constexpr int CHP = CH + 1;                 // K row pitch in chunks (odd)
  constexpr int EPC = 16 / ES;                // elements per 16-byte chunk
  constexpr int VTP = KC / EPC + 1;           // V^T row pitch in chunks (odd)
  constexpr int KL = KC * CH / ATT_THREADS;   // 16-byte loads per thread, tensor and chunk
  constexpr int NDT = D / 32;                 // 32-wide tiles of the head dimension
  constexpr int TPC = KC / 32;                // key tiles per chunk
  constexpr int RUNS = 32 / (2 * EPC);        // operand chunks per lane and 32-key tile in P.V
  constexpr int K_ROWS_PER_LOAD = ATT_THREADS / CH;
  constexpr int V_GROUPS_PER_LOAD = ATT_THREADS / (EPC * CH);

  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, rl = lane & 31, kg = lane >> 5;
  // consecutive indices stay on one XCD: the row groups and splits of a head share that XCD's L2
  const int n_wg = gridDim.x;
  const int idx = xcd_major(blockIdx.x, n_wg);
  const int split = idx % p.n_splits, qg = (idx / p.n_splits) % p.n_qgroups, h = idx / (p.n_splits * p.n_qgroups);
  const int wprt = 1 << p.wprt_log;           // waves that share a row tile, over different key tiles
  const int rt = wave >> p.wprt_log, ks = wave & (wprt - 1);
  const int row = qg * ATT_ROWS + rt * 32 + rl;

  extern __shared__ uint4 smem[];
  uint4* sK = smem;                           // [KC][CHP]
  uint4* sVT = smem + KC * CHP;               // [D][VTP]: V^T, element (d, key) at chunk key / EPC of row d

  // the wave's 32 query rows, as the B operand of S^T
  uint4 a[NCH];
  int blk_end_lane;  // block keys [0, blk_end_lane) are visible to this lane's row
  {
    const int m = min(row, p.m_rows - 1);
    const int g = m / p.n_q, j = m - g * p.n_q;
    const char* ptr = p.q.base + (int64_t)(h * p.group + g) * p.q.stride_head + (int64_t)j * p.q.stride_row;
#pragma unroll
    for (int i = 0; i < NCH; ++i) a[i] = ld16(ptr + (2 * i + kg) * 16);
    blk_end_lane = max(0, min(p.s_t, p.diag + j + 1));
  }
  // key ranges of this split in the two segments; the block range ends where the last row of the workgroup
  // stops seeing keys
  const int lo0 = min(split * p.keys_per_split, p.cache_len), hi0 = min(lo0 + p.keys_per_split, p.cache_len);
  int lo1 = 0, hi1 = 0;
  if (p.s_t > 0) {
    const int m0 = qg * ATT_ROWS, m1 = min(m0 + ATT_ROWS, p.m_rows) - 1;
    const int g0 = m0 / p.n_q, g1 = m1 / p.n_q;
    const int j_max = g0 == g1 ? m1 - g1 * p.n_q : p.n_q - 1;
    const int wg_end = max(0, min(p.s_t, p.diag + j_max + 1));
    lo1 = min(split * p.blk_keys_per_split, wg_end);
    hi1 = min(lo1 + p.blk_keys_per_split, wg_end);
  }

  const __amdgpu_buffer_rsrc_t ksrd0 = make_srd(p.k_cache + (int64_t)h * p.cache_stride_head, (uint32_t)p.cache_len * (uint32_t)p.row_bytes);
  const __amdgpu_buffer_rsrc_t vsrd0 = make_srd(p.v_cache + (int64_t)h * p.cache_stride_head, (uint32_t)p.cache_len * (uint32_t)p.row_bytes);
  const uint32_t kb_bytes = p.s_t > 0 ? (uint32_t)(p.s_t - 1) * (uint32_t)p.kb_stride_row + (uint32_t)p.row_bytes : 0u;
  const uint32_t vb_bytes = p.s_t > 0 ? (uint32_t)(p.s_t - 1) * (uint32_t)p.vb_stride_row + (uint32_t)p.row_bytes : 0u;
  const __amdgpu_buffer_rsrc_t ksrd1 = make_srd(p.k_blk + (int64_t)h * p.kb_stride_head, kb_bytes);
  const __amdgpu_buffer_rsrc_t vsrd1 = make_srd(p.v_blk + (int64_t)h * p.vb_stride_head, vb_bytes);
  // K: chunk tid % CH of row tid / CH (+ K_ROWS_PER_LOAD per load).  V: lane groups of EPC consecutive lanes
  // hold EPC consecutive keys at the same chunk, the shape the register transpose wants.
  const uint32_t k_row = tid / CH, k_col = tid % CH;
  const uint32_t v_i = tid % EPC, v_c = (tid / EPC) % CH, v_grp = tid / (EPC * CH);
  uint4 kpre[KL], vpre[KL];
  auto prefetch = [&](int seg, int kc0) {
    const __amdgpu_buffer_rsrc_t ksrd = seg ? ksrd1 : ksrd0, vsrd = seg ? vsrd1 : vsrd0;
    const uint32_t kstride = seg ? (uint32_t)p.kb_stride_row : (uint32_t)p.row_bytes;
    const uint32_t vstride = seg ? (uint32_t)p.vb_stride_row : (uint32_t)p.row_bytes;
#pragma unroll
    for (int u = 0; u < KL; ++u) {
      kpre[u] = buf_ld16(ksrd, (uint32_t)(kc0 + k_row + u * K_ROWS_PER_LOAD) * kstride + k_col * 16);
      const uint32_t key = (u * V_GROUPS_PER_LOAD + v_grp) * EPC + v_i;
      vpre[u] = buf_ld16(vsrd, (uint32_t)(kc0 + key) * vstride + v_c * 16);
    }
  };

  float m_ref = NEG_BIG, l_sum = 0.0f;
  f32x16 o[NDT];
#pragma unroll
  for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[dt][r] = 0.0f;

  int seg = lo0 < hi0 ? 0 : 1;
  int kc0 = seg ? lo1 : lo0;
  bool have = seg ? lo1 < hi1 : true;
  if (have) prefetch(seg, kc0);
  while (have) {
    lds_barrier();  // every wave has finished with the previous chunk
#pragma unroll
    for (int u = 0; u < KL; ++u) {
      sK[(k_row + u * K_ROWS_PER_LOAD) * CHP + k_col] = kpre[u];
      const uint4 t = DT == DT_BF16 ? transpose_8x8_b16(vpre[u], lane) : transpose_4x4_b32(vpre[u], lane);
      // the lane now holds head-dimension index v_c * EPC + v_i for the group's EPC keys
      store_vt<DT>(sVT + (v_c * EPC + v_i) * VTP, u * V_GROUPS_PER_LOAD + v_grp, t);
    }
    // the chunk after this one: the next of the segment, else the first of the block's keys
    int nseg = seg, nkc = kc0 + KC;
    bool nhave = nkc < (seg ? hi1 : hi0);
    if (!nhave && seg == 0 && lo1 < hi1) {
      nseg = 1;
      nkc = lo1;
      nhave = true;
    }
    if (nhave) prefetch(nseg, nkc);  // in flight while this chunk is worked on
    lds_barrier();

    const int k_hi = seg ? hi1 : hi0;
    const int lane_end = seg ? min(hi1, blk_end_lane) : hi0;  // end of the keys of this segment the lane's row sees
#pragma unroll 1
    for (int nt = ks; nt < TPC; nt += wprt) {
      const int kbase = kc0 + nt * 32;
      if (kbase >= k_hi) break;  // wave-uniform
      const int n_vis = lane_end - kbase;  // keys of this tile the lane's row sees (>= 32: all)
      if (!__any(n_vis > 0)) continue;     // the tile lies past the limit of every row of the wave
      f32x16 acc;
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
      const uint4* krow = sK + (size_t)(nt * 32 + rl) * CHP + kg;
#pragma unroll
      for (int i = 0; i < NCH; ++i) Mma<DT>::run(acc, krow[2 * i], a[i]);
      // hidden keys (past the end of the split or past the row's causal limit) weigh nothing, and a row that
      // sees no key of the tile keeps its state
      if (!__all(n_vis >= 32)) {
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] = acc_row(r, kg) < n_vis ? acc[r] : NEG_BIG;
      }
      float mx = acc[0];
#pragma unroll
      for (int r = 1; r < 16; ++r) mx = fmaxf(mx, acc[r]);
      mx = half_pair_max(mx);  // both halves of the wave use one reference per row
      mx = mx > NEG_BIG ? mx * p.scale2 : NEG_BIG;  // the reference lives in the scaled (log2) domain; scale2 > 0
      if (__any(mx > m_ref)) {
        const float m_new = fmaxf(m_ref, mx);
        const float alpha = fast_exp2(m_ref - m_new);
        l_sum *= alpha;
#pragma unroll
        for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
          for (int r = 0; r < 16; ++r) o[dt][r] *= alpha;
        m_ref = m_new;
      }
      // a row without a visible key so far subtracts nothing: its hidden logits give 2^(NEG_BIG * scale2) = 0
      const float m_sub = m_ref > NEG_BIG ? m_ref : 0.0f;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        acc[r] = fast_exp2(fmaf(acc[r], p.scale2, -m_sub));
        l_sum += acc[r];
      }
#pragma unroll
      for (int s = 0; s < RUNS; ++s) {
        uint4 pb;
        if (DT == DT_BF16) {
          pb = make_uint4(pack_bf16(acc[8 * s], acc[8 * s + 1]), pack_bf16(acc[8 * s + 2], acc[8 * s + 3]),
                          pack_bf16(acc[8 * s + 4], acc[8 * s + 5]), pack_bf16(acc[8 * s + 6], acc[8 * s + 7]));
        } else {
          pb = make_uint4(__float_as_uint(acc[4 * s]), __float_as_uint(acc[4 * s + 1]),
                          __float_as_uint(acc[4 * s + 2]), __float_as_uint(acc[4 * s + 3]));
        }
#pragma unroll
        for (int dt = 0; dt < NDT; ++dt) {
          const uint4* vrow = sVT + (size_t)(dt * 32 + rl) * VTP;
          uint4 va;
          if (DT == DT_BF16) {
            va = vrow[nt * 4 + 2 * s + kg];  // registers 8s .. 8s+7 are keys 16s + 4kg + (0..3) and the same + 8: see store_vt
          } else {
            va = vrow[nt * 8 + 2 * s + kg];  // registers 4s .. 4s+3 are keys 8s + 4kg + (0..3)
          }
          Mma<DT>::run(o[dt], va, pb);
        }
      }
    }
    seg = nseg;
    kc0 = nkc;
    have = nhave;
  }

  l_sum = half_pair_sum(l_sum);
  // several waves share a row tile over different key tiles: their states meet in LDS (rows padded by four
  // floats against bank conflicts) and leave as one partial per split
  constexpr int OP = D + 4;
  float* sO = reinterpret_cast<float*>(smem);                       // [8 waves][32 rows][OP]
  float2* sML = reinterpret_cast<float2*>(sO + ATT_WAVES * 32 * OP);  // [8 waves][32 rows]
  lds_barrier();  // the chunk buffers are free
  {
    float* dst = sO + (size_t)(wave * 32 + rl) * OP;
#pragma unroll
    for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4)
        *reinterpret_cast<float4*>(dst + dt * 32 + 8 * q4 + 4 * kg) =
            make_float4(o[dt][4 * q4], o[dt][4 * q4 + 1], o[dt][4 * q4 + 2], o[dt][4 * q4 + 3]);
    if (kg == 0) sML[wave * 32 + rl] = make_float2(m_ref, l_sum);
  }
  lds_barrier();
  const int n_rtw = ATT_WAVES >> p.wprt_log;  // row tiles of this workgroup
  for (int e = tid; e < n_rtw * 32 * (D / 4); e += ATT_THREADS) {
    const int d4 = e % (D / 4), rr = e / (D / 4);  // rr = row tile * 32 + row in tile
    const int row2 = qg * ATT_ROWS + rr;
    if (row2 >= p.m_rows) continue;
    const int w0 = (rr >> 5) << p.wprt_log, r2 = rr & 31;  // first wave of the tile
    float mx = NEG_BIG;
    for (int k = 0; k < wprt; ++k) mx = fmaxf(mx, sML[(w0 + k) * 32 + r2].x);
    float l = 0.0f;
    float4 acc = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    for (int k = 0; k < wprt; ++k) {
      const float2 ml = sML[(w0 + k) * 32 + r2];
      const float wgt = fast_exp2(ml.x - mx);
      const float4 ov = *reinterpret_cast<const float4*>(sO + (size_t)((w0 + k) * 32 + r2) * OP + d4 * 4);
      l = fmaf(ml.y, wgt, l);
      acc.x = fmaf(ov.x, wgt, acc.x);
      acc.y = fmaf(ov.y, wgt, acc.y);
      acc.z = fmaf(ov.z, wgt, acc.z);
      acc.w = fmaf(ov.w, wgt, acc.w);
    }
    const size_t at = ((size_t)h * p.n_parts + split) * p.m_rows + row2;
    if (d4 == 0) p.part_ml[at] = make_float2(mx, l);
    *reinterpret_cast<float4*>(p.part_o + at * D + d4 * 4) = acc;
  }
}

// The same pass for launches with more than four row tiles per KV head (window rows, whole blocks), arranged so that the
// matrix unit and the vector unit work at the same time and that every workgroup has the same work.
//   Pairs.  Waves w and w + 4 (one SIMD) take the row tiles i and n_tiles - 1 - i.  Row m = g n_q + j mirrors to the query
//   n_q - 1 - j, so under the causal mask of a whole block the two tiles see the block's first L and H keys with L + H the
//   same for all pairs.  The wave with fewer keys writes its result when the keys pass L and joins the other tile: from
//   then on the two waves take alternate 32-key tiles, and their states meet in LDS at the end.  (With
//   consecutive tiles in a workgroup a launch takes as long as the block's last rows: a 16k prefill of 32 heads in blocks
//   of 2048 rows took 169 us a block on average, with pairs 151.)
//   Tile loop.  Over long key ranges references are fixed, so that the output accumulators see nothing but matrix
//   instructions: there the tiles of a wave run on through a ring of four LDS stages in a fixed order of instructions
//   (`ring`).  Elsewhere two key tiles at a time, chunks alternating between two LDS stages; one barrier per chunk either
//   way, the next chunks arriving through async_ld16.  LDS addresses are kept per operand chunk (computed at each read they
//   cost 4 % of the time).
// Bound by the matrix unit, at the clock that power allows: 128k prefill, last block, 1136 -> 1249 TFLOP/s sustained with the
// ring (calls of 3690-3830 us -> 3500-3530; the loop alone on operands in LDS reaches 1326, and 1850 when they are zeros),
// window rows over 63 520 keys 149 -> 140 us.  By LDS reads it is bound to about the same: 16 KiB per wave and tile, a clock for
// 128 bytes.  In the ring's instance registers are short: what is needed only before and after the loops is computed from the
// thread's number there (with two registers in scratch memory a block of 1298 rows without a cache took 73.5 us instead of 71.1).
template <int DT>
__host__ __device__ constexpr int rows_chunk_keys() { return DT == DT_BF16 ? 128 : 64; }

// the order of V's 32-byte pieces by key: 16 lanes read four keys at one piece, 32 lanes at two neighbouring ones, and
// both sets are to lie in different banks
template <int CH>
__device__ __forceinline__ uint32_t v_swz(uint32_t key) { return CH == 8 ? key : 2 * key + (key >> 1); }

// Cache rows of a key range from which on its references are fixed (bf16).
constexpr int FIXED_KEYS = 320;
// ... from which on they pass through the ring before a block's own keys: 1024 rows over 455 and their block 47.7 us, with the
// ring 48.5, but block of 2048 over 1000 88.4 and 86.4.
constexpr int RING_KEYS = 512;

LKV_HD RowsShape rows_shape(const AttendParams& p) { return {p.m_rows, p.n_q, p.nq_magic, p.cache_len, p.s_t, p.diag}; }

// RING: with the ring (key ranges of at most FIXED_KEYS cache rows never enter it)
template <int DT, int D, bool RING>
__global__ __launch_bounds__(ATT_THREADS) void attend_rows_kernel(AttendParams p) {
  constexpr int ES = DT == DT_BF16 ? 2 : 4;
  constexpr int CH = D * ES / 16;             // 16-byte chunks per row
  constexpr int NCH = CH / 2;
  constexpr int KC = rows_chunk_keys<DT>();   // keys per LDS chunk
  constexpr int EPC = 16 / ES;                // elements per 16-byte chunk
  constexpr int VTP = KC / EPC + 1;           // V^T row pitch in chunks (odd)
  constexpr int KL = KC * CH / ATT_THREADS;   // 16-byte loads per thread, tensor and chunk
  constexpr int NDT = D / 32;                 // 32-wide tiles of the head dimension
  constexpr int TPC = KC / 32;                // key tiles per chunk
  constexpr int RUNS = 32 / (2 * EPC);        // operand chunks per lane and 32-key tile in P.V
  constexpr int ROWS_PER_LOAD = ATT_THREADS / CH;
  constexpr int V_GROUPS_PER_LOAD = ATT_THREADS / (EPC * CH);
  // Rows of K lie in LDS without padding (they arrive through async_ld16); chunk c of row r at position c ^ (r & KX), so
  // that consecutive rows of one operand chunk lie in different banks.
  constexpr int KX = CH < 16 ? CH - 1 : 15;
  // bf16: V stays key-major too and ds_read_b64_tr_b16 delivers it transposed; its 32-byte pieces are permuted by the
  // key (v_swz): a transposing read of four keys touches every bank once.  fp32 has no such read: V^T is built in
  // registers
  constexpr bool TR = DT == DT_BF16;
  constexpr int STAGE = KC * CH + (TR ? KC * CH : D * VTP);   // uint4 per LDS stage: K [KC][CH], then V [KC][CH] or V^T [D][VTP]
  static_assert(KL >= 1 && KL * ATT_THREADS == KC * CH, "chunk not a whole number of loads per thread");

  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, rl = lane & 31, kg = lane >> 5;
  // The first n_full workgroups take all keys of their rows, the others the n_splits key ranges of the last n_cut row
  // groups.  Consecutive indices stay on one XCD: the row groups and splits of a head share that XCD's L2
  const bool full = (int)blockIdx.x < p.n_full;
  const int idx = full ? xcd_major(blockIdx.x, p.n_full) : xcd_major(blockIdx.x - p.n_full, p.n_cut * p.n_splits);
  const int n_splits = full ? 1 : p.n_splits, split = full ? 0 : idx % n_splits, cut_wg = full ? 0 : idx / n_splits;
  const int wg = full ? idx : p.n_full + cut_wg, pg = wg % p.n_qgroups, h = wg / p.n_qgroups;
  const bool direct = n_splits == 1;

  const int n_tiles = (p.m_rows + 31) >> 5, n_pairs = (n_tiles + 1) >> 1;
  const RowsShape shape = rows_shape(p);
  const int upper = __builtin_amdgcn_readfirstlane(wave >> 2);  // the pair's wave whose tile sees more keys
  const int pr = pg * 4 + (__builtin_amdgcn_readfirstlane(wave) & 3);
  const bool present = pr < n_pairs;
  int t_lo = min(pr, n_pairs - 1), t_hi = n_tiles - 1 - t_lo;
  const bool single = t_lo == t_hi;           // the middle tile of an odd number: both waves work on it
  int end_lo = rows_tile_end(shape, t_lo), end_hi = rows_tile_end(shape, t_hi);
  if (end_lo > end_hi) {
    int t = t_lo; t_lo = t_hi; t_hi = t;
    t = end_lo; end_lo = end_hi; end_hi = t;
  }
  // this split's keys
  int lo0, hi0, lo1, hi1;
  {
    const RowsCut rc = rows_cut(shape, pg, n_splits);
    auto cut = [&](int s, int& c, int& b) {  // the start of split s in the two segments, multiples of 32 (or their ends)
      const int t = s * rc.share, x = t <= rc.both ? t : rc.both + 2 * (t - rc.both);
      c = min(x, p.cache_len);
      b = s >= n_splits ? rc.end : min(max(x - p.cache_len, 0) & ~31, rc.end);
    };
    cut(split, lo0, lo1);
    cut(split + 1, hi0, hi1);
    if (split + 1 >= n_splits) hi0 = p.cache_len;
  }

  extern __shared__ uint4 smem[];

  // the rows of the wave's current tile, as the B operand of S^T
  uint4 a[NCH];
  int blk_end_lane;  // block keys [0, blk_end_lane) are visible to this lane's row
  auto fetch_rows = [&](int t) {
    const int tid_r = fresh(tid), row = t * 32 + (tid_r & 31), m = min(RING ? row : fresh(row), p.m_rows - 1);
    int j;
    const int g = div_rem(m, p.n_q, p.nq_magic, &j);
    const char* ptr = p.q.base + (int64_t)(h * p.group + g) * p.q.stride_head + (int64_t)j * p.q.stride_row + (tid_r >> 5 & 1) * 16;
#pragma unroll
    for (int i = 0; i < NCH; ++i) a[i] = ld16(ptr + 2 * i * 16);
    blk_end_lane = max(0, min(p.s_t, p.diag + j + 1));
  };
  auto rows_landed = [&]() {
#pragma unroll
    for (int i = 0; i < NCH; ++i) landed(a[i]);
  };
  auto load_rows = [&](int t) {
    fetch_rows(t);
    rows_landed();
  };

  // the segments: the cache (0) and the block's own rows (1)
  const uint32_t kb_bytes = p.s_t > 0 ? (uint32_t)(p.s_t - 1) * (uint32_t)p.kb_stride_row + (uint32_t)p.row_bytes : 0u;
  const uint32_t vb_bytes = p.s_t > 0 ? (uint32_t)(p.s_t - 1) * (uint32_t)p.vb_stride_row + (uint32_t)p.row_bytes : 0u;
  const char* k_base0 = p.k_cache + (int64_t)h * p.cache_stride_head;
  const char* v_base0 = p.v_cache + (int64_t)h * p.cache_stride_head;
  const char* k_base1 = p.k_blk + (int64_t)h * p.kb_stride_head;
  const char* v_base1 = p.v_blk + (int64_t)h * p.vb_stride_head;
  const uint32_t c_bytes = (uint32_t)p.cache_len * (uint32_t)p.row_bytes;
  const uint32_t lds0 = lds_offset(smem);
  // chunk lane % CH of row ld_row (+ ROWS_PER_LOAD per load)
  const uint32_t ld_row = wave * (64 / CH) + lane / CH, ld_pos = lane % CH;
  const uint32_t k_col = (ld_pos ^ (ld_row & KX)) * 16, v_col = (ld_pos ^ (2 * v_swz<CH>(ld_row & 3))) * 16;
  const uint32_t v_i = tid % EPC, v_c = (tid / EPC) % CH, v_grp = tid / (EPC * CH);
  uint4 vpre[TR ? 1 : KL];
  // bf16 rows of 256 bytes: the first waves bring the keys, and tiles against following references pass in a fixed order.
  // Rows of 128 bytes have half the loads and half the products to put anything beside; both cost there (block of 4096 rows
  // over 64 cache rows 124.4 us, 122.8 with all waves loading, 122.2 with the compiler's order too; 2048 rows over 3000 85.1,
  // 84.5, 83.8; 64 rows over 31 681 32.2, 31.7, 31.7).
  constexpr bool WIDE = TR && CH == 16;
  constexpr int SHARE = WIDE ? 2 : 1;  // of the loads that a loading wave takes
  // Starts the loads of a chunk into a stage.  Rows past the segment's last one repeat it (they weigh nothing).  The
  // asynchronous loads come from the first wave of every SIMD: 64 KiB keep the address unit busy for a thousand clocks, and
  // while the first waves wait for it the second ones have the SIMDs to themselves.  From all waves, behind the barrier, both
  // stood still for it, and so they did with the loads spread over the tiles' steps.  (Here block of 4096 rows over 64 cache
  // rows 186 -> 181 us, in the ring last block of a 128k prefill 3580 -> 3540, window rows over 63 520 keys 135.2 -> 134.5.)
  auto prefetch = [&](int seg, int kc0, int stage) {
    const srd_words ksrd = make_srd_words(seg ? k_base1 : k_base0, seg ? kb_bytes : c_bytes);
    const srd_words vsrd = make_srd_words(seg ? v_base1 : v_base0, seg ? vb_bytes : c_bytes);
    const uint32_t kstride = seg ? (uint32_t)p.kb_stride_row : (uint32_t)p.row_bytes;
    const uint32_t vstride = seg ? (uint32_t)p.vb_stride_row : (uint32_t)p.row_bytes;
    const uint32_t rows = (uint32_t)(seg ? p.s_t : p.cache_len);
    const uint32_t dst = lds0 + stage * (STAGE * 16) + __builtin_amdgcn_readfirstlane(wave) * 1024;
    const uint32_t r0 = fresh(ld_row);
    if (WIDE && upper) return;
    // (fp32: every thread has its loads of V besides)
    constexpr int N = SHARE * KL, ROWS = ROWS_PER_LOAD * KL / N, BYTES = ATT_THREADS * 16 * KL / N;
    if (kc0 + KC <= (int)rows) {
      const uint32_t k_off = r0 * kstride + k_col, v_off = r0 * vstride + v_col;
#pragma unroll
      for (int u = 0; u < N; ++u) {
        const uint32_t row = kc0 + u * ROWS;
        async_ld16(ksrd, k_off, row * kstride, dst + u * BYTES);
        if (TR) async_ld16(vsrd, v_off, row * vstride, dst + KC * CH * 16 + u * BYTES);
      }
    } else {
#pragma unroll 1
      for (int u = 0; u < N; ++u) {
        const uint32_t row = min((uint32_t)kc0 + r0 + u * ROWS, rows - 1u);
        async_ld16(ksrd, row * kstride + k_col, 0u, dst + u * BYTES);
        if (TR) async_ld16(vsrd, row * vstride + v_col, 0u, dst + KC * CH * 16 + u * BYTES);
      }
    }
    if (!TR) {
      const __amdgpu_buffer_rsrc_t vs = make_srd(seg ? v_base1 : v_base0, seg ? vb_bytes : c_bytes);
#pragma unroll
      for (int u = 0; u < KL; ++u) {
        const uint32_t key = (u * V_GROUPS_PER_LOAD + v_grp) * EPC + v_i;
        vpre[u] = buf_ld16(vs, (uint32_t)(kc0 + key) * vstride + v_c * 16);
      }
    }
  };
  // Completes them (fp32: V^T is written here).
  auto land = [&](int stage) {
    if (!TR) {
      uint4* sV = smem + (size_t)stage * STAGE + KC * CH;
#pragma unroll
      for (int u = 0; u < KL; ++u)
        store_vt<DT>(sV + (v_c * EPC + v_i) * VTP, u * V_GROUPS_PER_LOAD + v_grp, transpose_4x4_b32(vpre[u], lane));
    }
    async_wait();
  };
  // Transposing read of V (bf16).  Within 16 lanes, lane i hands in the address of 4 consecutive 16-bit values and
  // lane 4c + e receives value e of lanes c, c + 4, c + 8, c + 12.  Lane i points at key (i >> 2) of a run of four
  // keys and head-dimension offset 4 (i & 3), so lane l of the sixteen receives the four keys at head-dimension
  // offset l: the A operand of O^T += V^T P^T.  Byte offset of this lane's piece within a V stage, for key 0 of the
  // tile's first 16-key block and head-dimension tile 0:
  // LDS addresses of a lane's pieces for a tile in the first rows of a stage: K, to be xored with 32 i for operand chunk
  // pair i, and V, to be xored with 64 dt for head-dimension tile dt (rows are powers of two, so rows are added and
  // positions within them xored)
  const uint32_t k_at = lds0 + rl * (CH * 16) + ((kg ^ (rl & KX)) * 16);
  const uint32_t v_at = TR ? lds0 + KC * CH * 16 + (4 * kg + ((lane & 15) >> 2)) * CH * 16 + (lane & 3) * 8 +
                                 (((2 * ((lane >> 4) & 1)) ^ (2 * v_swz<CH>((lane & 15) >> 2))) * 16)
                           : lds0 + KC * CH * 16 + rl * (VTP * 16) + kg * 16;
  constexpr uint32_t K_TILE = 32 * CH * 16, V_TILE = TR ? 32 * CH * 16 : 32 / EPC * 16;  // bytes from one 32-key tile to the next
  // the chunk after (seg, kc0): the next of the segment, else the first of the block's keys
  auto advance = [&](int& seg, int& kc0) -> bool {
    kc0 += KC;
    if (kc0 < (seg ? hi1 : hi0)) return true;
    if (seg == 0 && lo1 < hi1) {
      seg = 1;
      kc0 = lo1;
      return true;
    }
    return false;
  };
  auto load_k = [&](uint32_t at, uint4* kf) {  // a key tile's operand chunks
    at = opaque(at);
#pragma unroll
    for (int i = 0; i < NCH; ++i) kf[i] = lds_ld16(at ^ (32 * i));
  };
  auto logits = [&](const uint4* kf, f32x16& acc) {
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
#pragma unroll
    for (int i = 0; i < NCH; ++i) Mma<DT>::run(acc, kf[i], a[i]);
  };

  float m_ref, l_sum;
  f32x16 o[NDT];
  auto clear = [&]() {
    m_ref = NEG_BIG;
    l_sum = 0.0f;
#pragma unroll
    for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
      for (int r = 0; r < 16; ++r) o[dt][r] = 0.0f;
  };
  auto load_v = [&](uint32_t vat, uint4* vf) {  // fp32
#pragma unroll
    for (int s = 0; s < RUNS; ++s)
#pragma unroll
      for (int dt = 0; dt < NDT; ++dt) vf[s * NDT + dt] = lds_ld16(vat + dt * (32 * VTP * 16) + 2 * s * 16);  // registers 4s .. 4s+3 are keys 8s + 4kg + (0..3)
  };
  auto load_v_tr = [&](const uint32_t* vx, uint32_t off, uint4* vf) {  // bf16
#pragma unroll
    for (int s = 0; s < RUNS; ++s)
#pragma unroll
      for (int dt = 0; dt < NDT; ++dt) {
        // registers 8s .. 8s+3 of the logits are keys 16s + 4kg + (0..3), registers 8s+4 .. 8s+7 the same + 8
        const uint32_t at = vx[dt] + off + 16 * s * CH * 16;
        const uint2 lo = ds_read_tr16(at), hi = ds_read_tr16(at + 8 * CH * 16);
        vf[s * NDT + dt] = make_uint4(lo.x, lo.y, hi.x, hi.y);
      }
  };
  auto weigh = [&](const f32x16& acc, const uint4* vf) {  // O^T += V^T P^T
#pragma unroll
    for (int s = 0; s < RUNS; ++s) {
      uint4 pb;
      if (DT == DT_BF16) {
        pb = make_uint4(pack_bf16(acc[8 * s], acc[8 * s + 1]), pack_bf16(acc[8 * s + 2], acc[8 * s + 3]),
                        pack_bf16(acc[8 * s + 4], acc[8 * s + 5]), pack_bf16(acc[8 * s + 6], acc[8 * s + 7]));
      } else {
        pb = make_uint4(__float_as_uint(acc[4 * s]), __float_as_uint(acc[4 * s + 1]),
                        __float_as_uint(acc[4 * s + 2]), __float_as_uint(acc[4 * s + 3]));
      }
#pragma unroll
      for (int dt = 0; dt < NDT; ++dt) Mma<DT>::run(o[dt], vf[s * NDT + dt], pb);
    }
  };
  auto finite = [&]() -> bool {  // the lane's sum and outputs below 2^127
    uint32_t top = __float_as_uint(l_sum) << 1;
#pragma unroll
    for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
      for (int r = 0; r < 16; ++r) top = max(top, __float_as_uint(o[dt][r]) << 1);
    return top < 0xfe000000u;
  };
  // Moves a sum's growth past one into the reference: states are merged and divided as if the reference had been there.
  auto settle = [&]() {
    const float l = half_pair_max(l_sum);  // one reference for both halves
    const int e = l > 1.0f ? __builtin_amdgcn_frexp_expf(l) : 0;
    m_ref += (float)e;
    l_sum = __builtin_amdgcn_ldexpf(l_sum, -e);
#pragma unroll
    for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
      for (int r = 0; r < 16; ++r) o[dt][r] = __builtin_amdgcn_ldexpf(o[dt][r], -e);
  };
  // The result of tile t from the wave's complete state: with one split out = O / l and lse = (m + log2 l) ln 2 (a row
  // that saw no key gives zero and -inf), else the split's partial (reference, sum, unnormalised output).  A lane holds 16
  // bytes of every 32 of its row; groups of four lanes exchange them so that a store instruction writes whole 128-byte
  // lines of eight rows (with 32-byte pieces of
  // 32 rows the 33 MB of 65536 rows took 3.6 us longer).
  // the ring's instance keeps nothing of it through the loops (the other one has the registers: 11.85 -> 11.7 us for 64 rows a
  // head over 74 keys)
  auto late = [&]() { return RING ? fresh(tid) : tid; };
  auto write_tile = [&](int t) {
    const int tid_w = late(), wave = tid_w >> 6, lane = tid_w & 63, rl = lane & 31, kg = lane >> 5;
    const int row = RING ? t * 32 + rl : fresh(t * 32 + rl);
    const float l = half_pair_sum(l_sum);
    float scale = 1.0f, *dst;
    if (direct) {
      const size_t at = (size_t)h * p.m_rows + row;
      scale = l > 0.0f ? 1.0f / l : 0.0f;
      if (kg == 0 && row < p.m_rows) p.out_lse[at] = l > 0.0f ? lse_log2(m_ref, l) * 0.6931471805599453f : -__builtin_inff();
      dst = p.out + (size_t)h * p.m_rows * D;
    } else {
      // [cut row groups][splits][256 rows: the pairs in order, of each the tile with the lower number first]
      const size_t at = ((size_t)cut_wg * n_splits + split) * ATT_ROWS + ((wave & 3) * 2 + (t != pr)) * 32;
      if (kg == 0) p.part_ml[at + rl] = make_float2(m_ref, l);
      dst = p.part_o + at * D - (size_t)t * 32 * D;
    }
    const int row4 = row & ~3;
    dst += (int64_t)row4 * D + 8 * (rl & 3) + 4 * kg;
#pragma unroll
    for (int dt = 0; dt < NDT; ++dt) {
      uint4 x[4];  // component u of the lane's four pieces, then of its piece of four rows
#pragma unroll
      for (int u = 0; u < 4; ++u)
        x[u] = transpose_4x4_b32(make_uint4(__float_as_uint(o[dt][u] * scale), __float_as_uint(o[dt][4 + u] * scale),
                                            __float_as_uint(o[dt][8 + u] * scale), __float_as_uint(o[dt][12 + u] * scale)), lane);
      const uint4 piece[4] = {make_uint4(x[0].x, x[1].x, x[2].x, x[3].x), make_uint4(x[0].y, x[1].y, x[2].y, x[3].y),
                              make_uint4(x[0].z, x[1].z, x[2].z, x[3].z), make_uint4(x[0].w, x[1].w, x[2].w, x[3].w)};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if (row4 + e >= p.m_rows) continue;
        if (direct) st16_stream(dst + (size_t)e * D + dt * 32, piece[e]);
        else *reinterpret_cast<uint4*>(dst + (size_t)e * D + dt * 32) = piece[e];
      }
    }
  };

  // In bf16 a row's reference follows the maximum, tile by tile: the dominant key's probability is then a power of two and
  // its bf16 exact, while against another reference its rounding (up to 2^-8) goes into the output whole.  But where the
  // key range has more than FIXED_KEYS cache rows, and in fp32, the reference over them is fixed: the row's maximum over the
  // first tile of keys that it sees, plus HEADROOM (what a row sees is a prefix of the keys: a row that sees none of a
  // wave's first tile sees none of the others).  Each logit then costs an fma, an exponential and an add, and the output
  // accumulators nothing but matrix instructions.
  // Measured: following costs 11 % over long ranges (window rows over 63 520 keys 147 -> 164 us, last block of a 128k
  // prefill 3.71 -> 4.14 ms), 9 % over short ones (256 rows over 8000 keys, 288 a range: 28.2 -> 30.8 us) and over the
  // block's own keys 3.4 % of a 16k prefill in blocks of 2048 (1330 -> 1375 us).  The line: up to there a fixed reference
  // is the worse the longer the range (the first tile holds the maximum of fewer rows; 288 keys 1.6e-3 of the output
  // against 2e-4), past it its error no longer changes.
  // Sums or outputs that overflow against a fixed reference (from about a logit 145 above the first tile's on, in powers
  // of two) make the workgroup repeat the pass with the exact maxima, which a sweep over the keys finds first.  (One
  // workgroup in a round that repeats it costs three times the round; keys whose lengths spread by e^0.5 reach 140.)
  constexpr bool BF16 = DT == DT_BF16;
  const bool fixed = !BF16 || hi0 - lo0 > FIXED_KEYS;
  int* redo = reinterpret_cast<int*>(smem + (size_t)2 * STAGE);  // one word behind the two stages
  if (tid == 0) *redo = 0;  // ordered before the writes after the first pass by the barriers in between
  // position in the split's chunks
  int seg, kc0, nseg, nkc, cur;
  bool have, nhave;
  auto start = [&](int from) {  // the first chunk's loads, cache rows from `from` on
    seg = from < hi0 ? 0 : 1;
    kc0 = seg ? lo1 : from;
    have = seg ? lo1 < hi1 : true;
    nseg = seg;
    nkc = kc0;
    nhave = false;
    cur = 0;
    if (have) {
      prefetch(seg, kc0, 0);
      nhave = advance(nseg, nkc);
    }
  };
  auto next = [&]() {  // on to the next chunk
    have = nhave;
    if (have) {
      land(cur ^ 1);
      seg = nseg;
      kc0 = nkc;
      nhave = advance(nseg, nkc);
      cur ^= 1;
      lds_barrier();
    }
  };
  auto hide = [&](f32x16& acc, int n_vis) {  // hidden keys (past the end of the split or the row's causal limit) weigh nothing
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = acc_row(r, 0) < n_vis - 4 * kg ? acc[r] : NEG_BIG;
  };
  auto maximum = [&](uint32_t at, int n_vis) {  // of a tile's visible logits, in the scaled (log2) domain; scale2 > 0
    f32x16 acc;
    uint4 kf[NCH];
    load_k(at, kf);
    logits(kf, acc);
    hide(acc, n_vis);
    float mx = acc[0];
#pragma unroll
    for (int r = 1; r < 16; ++r) mx = fmaxf(mx, acc[r]);
    mx = half_pair_max(mx);  // both halves of the wave use one reference per row
    return mx > NEG_BIG ? mx * p.scale2 : NEG_BIG;
  };
  bool joined;  // the pair's waves share the upper tile
  float ref_own = NEG_BIG, ref_join = NEG_BIG;  // the second pass's references for the wave's own tile and the shared one
  // The wave's key tiles in a chunk are nt0, nt0 + 1, ..., up to the last key that some row sees; sharing waves take half a
  // chunk each.
  int nt0;
  // LDS addresses of the lane's operand chunks in the wave's first tile of the current chunk (bf16; kept and moved from
  // stage to stage: computed where they are used they cost a vector instruction per LDS read)
  uint32_t kx[NCH], vx[NDT];
  auto place = [&]() {
    nt0 = joined && !upper ? TPC / 2 : 0;
#pragma unroll
    for (int i = 0; i < NCH; ++i) kx[i] = opaque((k_at + cur * (STAGE * 16) + nt0 * K_TILE) ^ (32 * i));
#pragma unroll
    for (int dt = 0; dt < NDT; ++dt) vx[dt] = opaque((v_at + cur * (STAGE * 16) + nt0 * V_TILE) ^ (64 * dt));
  };
  // Long ranges of cache rows against fixed references (bf16): a ring of four stages of 64 keys, each with its K and V.  The
  // tiles of a wave run on across the chunks: the products of a tile with the keys stand beside the exponentials of the
  // tile before, those with the values beside the next exponents.  One barrier per chunk tells that the next chunk has landed
  // and that the one before has been left.
  constexpr int RC = 64;                                     // keys per ring stage
  constexpr uint32_t R_V = RC * CH * 16, R_STAGE = 2 * R_V;  // bytes of K in a stage, and of K and V
  constexpr int R_LOADS = SHARE * RC * CH / ATT_THREADS;     // per loading thread, tensor and chunk
  // (not in the workgroup whose waves share the middle tile of an odd number from the start)
  const bool middle = (n_tiles & 1) && pg == (n_pairs - 1) / 4;
  const int ring_keys = BF16 && RING && fixed && !middle ? (hi0 - lo0) & ~(2 * RC - 1) : 0;
  const int n_ring = ring_keys / RC;
  auto ring_prefetch = [&](int c) {
    if (WIDE && upper) return;
    const srd_words ksrd = make_srd_words(k_base0, c_bytes), vsrd = make_srd_words(v_base0, c_bytes);
    const uint32_t r0 = fresh(ld_row) * (uint32_t)p.row_bytes, src = (uint32_t)(lo0 + c * RC) * (uint32_t)p.row_bytes;
    const uint32_t dst = lds0 + (c & 3) * R_STAGE + __builtin_amdgcn_readfirstlane(wave) * 1024;
#pragma unroll
    for (int u = 0; u < R_LOADS; ++u) {
      async_ld16(ksrd, r0 + k_col, src + u * (ROWS_PER_LOAD / SHARE) * (uint32_t)p.row_bytes, dst + u * (ATT_THREADS * 16 / SHARE));
      async_ld16(vsrd, r0 + v_col, src + u * (ROWS_PER_LOAD / SHARE) * (uint32_t)p.row_bytes, dst + R_V + u * (ATT_THREADS * 16 / SHARE));
    }
  };
  auto ring = [&](bool has_ref) {
    constexpr int AHEAD = NCH / 2;  // operands read ahead of the matrix instructions
    constexpr int PER = 16 / NCH;   // logits per step
    uint32_t kr[NCH], vr[NDT];
#pragma unroll
    for (int i = 0; i < NCH; ++i) kr[i] = opaque(k_at ^ (32 * i));
#pragma unroll
    for (int dt = 0; dt < NDT; ++dt) vr[dt] = opaque((v_at ^ (64 * dt)) - KC * CH * 16 + R_V);
    f32x16 x, nxt;  // a tile's exponents, the next one's logits
    uint4 kf[AHEAD], vf[AHEAD];
    // tile t of the four that two stages hold
    auto read_k = [&](int t, int i) { kf[i % AHEAD] = lds_ld16(kr[i], (t >> 1) * R_STAGE + (t & 1) * K_TILE); };
    auto read_v = [&](int t, int i) {
      // registers 8s .. 8s+3 of the logits are keys 16s + 4kg + (0..3), registers 8s+4 .. 8s+7 the same + 8
      const uint32_t at = vr[i % NDT] + (t >> 1) * R_STAGE + (t & 1) * V_TILE + 16 * (i / NDT) * CH * 16;
      const uint2 lo = ds_read_tr16(at), hi = ds_read_tr16(at + 8 * CH * 16);
      vf[i % AHEAD] = make_uint4(lo.x, lo.y, hi.x, hi.y);
    };
    uint32_t move = 2 * R_STAGE;  // to the other two stages
    float m_sub;
    auto unit = [&](int t) {
      uint4 pb[2];
#pragma unroll
      for (int r = 0; r < 16; ++r) nxt[r] = 0.0f;
#pragma unroll
      for (int i = 0; i < NCH; ++i) {
        Mma<DT>::run(nxt, kf[i % AHEAD], a[i]);
#pragma unroll
        for (int r = i * PER; r < (i + 1) * PER; ++r) {
          x[r] = fast_exp2(x[r]);
          l_sum += x[r];
        }
        if (i + AHEAD < NCH) read_k((t + 1) & 3, i + AHEAD);
        else read_v(t, i + AHEAD - NCH);
        if (i == NCH / 2 - 1 || i == NCH - 1) {
          const int s = i / (NCH / 2);
          pb[s] = make_uint4(pack_bf16(x[8 * s], x[8 * s + 1]), pack_bf16(x[8 * s + 2], x[8 * s + 3]),
                             pack_bf16(x[8 * s + 4], x[8 * s + 5]), pack_bf16(x[8 * s + 6], x[8 * s + 7]));
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      if (t == 2)  // the keys of the next tile but one lie in the other stages
#pragma unroll
        for (int i = 0; i < NCH; ++i) kr[i] = opaque(kr[i] + move);
#pragma unroll
      for (int i = 0; i < NCH; ++i) {
        Mma<DT>::run(o[i % NDT], vf[i % AHEAD], pb[i / NDT]);  // O^T += V^T P^T
        if (i + AHEAD < NCH) read_v(t, i + AHEAD);
        else read_k((t + 2) & 3, i + AHEAD - NCH);
        if (i > 0)  // the last product with the keys takes a step to arrive
#pragma unroll
          for (int r = (i - 1) * 16 / (NCH - 1); r < i * 16 / (NCH - 1); ++r) x[r] = fmaf(nxt[r], p.scale2, -m_sub);
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(4 * R_LOADS) : "memory");
    lds_barrier();
    if (present) {
#pragma unroll
      for (int r = 0; r < 16; ++r) nxt[r] = 0.0f;
#pragma unroll
      for (int i = 0; i < NCH; ++i) {
        kf[0] = lds_ld16(kr[i]);
        Mma<DT>::run(nxt, kf[0], a[i]);
      }
      if (!has_ref) {
        float mx = nxt[0];
#pragma unroll
        for (int r = 1; r < 16; ++r) mx = fmaxf(mx, nxt[r]);
        mx = half_pair_max(mx);
        m_ref = mx > NEG_BIG ? fmaf(mx, p.scale2, HEADROOM) : NEG_BIG;
      }
      m_sub = m_ref > NEG_BIG ? m_ref : 0.0f;
#pragma unroll
      for (int r = 0; r < 16; ++r) x[r] = fmaf(nxt[r], p.scale2, -m_sub);
#pragma unroll
      for (int i = 0; i < AHEAD; ++i) read_k(1, i);
    }
#pragma unroll 1
    for (int c = 0; c < n_ring; c += 2) {
#pragma unroll
      for (int half = 0; half < 2; ++half) {
        if (c + half + 2 < n_ring) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * R_LOADS) : "memory");
        else async_wait();
        lds_barrier();
        if (present) unit(2 * half);
        if (c + half + 3 < n_ring) ring_prefetch(c + half + 3);  // between two tiles: behind the barrier both waves of a SIMD stand still for it (2 - 3 %)
        if (present) unit(2 * half + 1);
      }
#pragma unroll
      for (int dt = 0; dt < NDT; ++dt) vr[dt] = opaque(vr[dt] + move);
      move = -move;
    }
    lds_barrier();  // every wave has left the stages
  };
#pragma unroll 1
  for (int pass = 0;; ++pass) {
    bool has_ref = pass != 0, bad = false;
    if (ring_keys) {
      for (int c = 0; c < 3; ++c) ring_prefetch(c);
      load_rows(upper ? t_hi : t_lo);
      clear();
      if (pass) m_ref = ref_own;
      ring(has_ref);
      has_ref = true;
      start(lo0 + ring_keys);
      joined = false;
      place();
    } else {
      start(lo0);
      joined = single && have;
      place();
      load_rows(upper || single ? t_hi : t_lo);
      clear();
      if (pass) m_ref = ref_own;
    }
    if (have) {
      land(0);
      lds_barrier();
    }
    // A loop for fixed references, then one for those that follow the maximum (fp32: one for each segment): in a loop for
    // both, what the second kind needs costs the first registers.
#pragma unroll
    for (int kind = 0; kind < 2; ++kind) {
      const bool follows = kind == 1 && BF16;
      while (have && (kind == 1 || (seg == 0 && fixed))) {
        if (nhave) prefetch(nseg, nkc, cur ^ 1);  // in flight while this chunk is worked on; every wave left that stage before the barrier
        if (kind && seg && !joined && kc0 >= end_lo) {
          joined = true;
          if (!upper) {
            bad = !finite();
            settle();
            fetch_rows(t_hi);  // in front of the stores, whose way to the memory it would wait for
            if (present) write_tile(t_lo);
            rows_landed();
            clear();
            place();
            has_ref = pass != 0;
            if (pass) m_ref = ref_join;
          }
        }
        const int wave_end = kind && seg ? min(hi1, upper || joined ? end_hi : end_lo) : hi0;
        int left = present ? min(min(max((wave_end - kc0 + 31) >> 5, 0), TPC) - nt0, joined ? TPC / 2 : TPC) : 0;
        const int lane_end = kind && seg ? min(hi1, blk_end_lane) : hi0;  // end of the keys of this segment the lane's row sees
        const int n_vis = lane_end - (kc0 + nt0 * 32);  // keys from the wave's first on that the lane's row sees
        const bool whole = kind ? __all(n_vis >= KC - nt0 * 32) : n_vis >= KC - nt0 * 32;
        if (left > 0 && !has_ref && !follows) {
          has_ref = true;
          m_ref = maximum(k_at + cur * (STAGE * 16) + nt0 * K_TILE, n_vis);
          m_ref += m_ref > NEG_BIG ? HEADROOM : 0.0f;
        }
        // a row without a visible key subtracts nothing: its hidden logits give 2^(NEG_BIG * scale2) = 0
        float m_sub = m_ref > NEG_BIG ? m_ref : 0.0f;
        auto soft = [&](f32x16& acc) {
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            acc[r] = fast_exp2(fmaf(acc[r], p.scale2, -m_sub));
            l_sum += acc[r];
          }
        };
        uint32_t moved = 0;  // of the LDS addresses within the chunk
        if (BF16) {
          if (!follows) {
            // two key tiles: the exponentials of one run beside the other's products
#pragma unroll
            for (int T = 0; T < TPC; T += 2) {
              if (left <= T) break;
              const int vis = n_vis - T * 32;
              f32x16 acc0, acc1;
              uint4 ka[NCH], kb[NCH], va[RUNS * NDT], vb[RUNS * NDT];
#pragma unroll
              for (int i = 0; i < NCH; ++i) ka[i] = lds_ld16(kx[i] + T * K_TILE);
#pragma unroll
              for (int i = 0; i < NCH; ++i) kb[i] = lds_ld16(kx[i] + (T + 1) * K_TILE);
              logits(ka, acc0);
              if (!whole) hide(acc0, vis);
              load_v_tr(vx, T * V_TILE, va);
              logits(kb, acc1);
              soft(acc0);
              if (!whole) hide(acc1, vis - 32);
              load_v_tr(vx, (T + 1) * V_TILE, vb);
              weigh(acc0, va);
              soft(acc1);
              weigh(acc1, vb);
            }
          } else if constexpr (!WIDE) {
            auto raise = [&](const f32x16& acc) {  // the reference, to the row's maximum in a tile
              float mx = acc[0];
#pragma unroll
              for (int r = 1; r < 16; ++r) mx = fmaxf(mx, acc[r]);
              mx = half_pair_max(mx);
              const float m_new = mx > NEG_BIG ? fmaxf(m_ref, fmaf(mx, p.scale2, HEADROOM)) : m_ref;
              if (__any(m_new > m_ref && l_sum > 0.0f)) {  // nothing to rescale before the first keys
                const float f = fast_exp2(m_ref - m_new);
                l_sum *= f;
#pragma unroll
                for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
                  for (int r = 0; r < 16; ++r) o[dt][r] *= f;
              }
              m_ref = m_new;
              m_sub = m_new > NEG_BIG ? m_new : 0.0f;
            };
#pragma unroll
            for (int T = 0; T < TPC; T += 2) {
              if (left <= T) break;
              f32x16 acc0, acc1;
              uint4 kf[NCH], vf[RUNS * NDT];
#pragma unroll
              for (int i = 0; i < NCH; ++i) kf[i] = lds_ld16(kx[i] + T * K_TILE);
              logits(kf, acc0);
#pragma unroll
              for (int i = 0; i < NCH; ++i) kf[i] = lds_ld16(kx[i] + (T + 1) * K_TILE);
              logits(kf, acc1);
              if (!whole) {
                hide(acc0, n_vis - T * 32);
                hide(acc1, n_vis - T * 32 - 32);
              }
              load_v_tr(vx, T * V_TILE, vf);
              raise(acc0);
              soft(acc0);
              weigh(acc0, vf);
              load_v_tr(vx, (T + 1) * V_TILE, vf);
              raise(acc1);
              soft(acc1);
              weigh(acc1, vf);
            }
          } else {
            // The products of a tile with the keys beside the exponentials of the tile before, those with the values beside
            // the maximum and the next exponents; operands are read four matrix instructions ahead (in the compiler's order
            // every product with the keys waited for its own read; 16k prefill in blocks of 2048 rows 1385 -> 1372 us).
            // Bound by issue: of some 1450 clocks per wave and two tiles 520 go into rescaling the output, which some row of
            // 32 asks for at most tiles.
            constexpr int AHEAD = 4, HALF = NCH / 2;
            static_assert(NCH == RUNS * NDT || !BF16, "as many products with the values as with the keys");
            f32x16 x, nxt;
            uint4 kf[AHEAD], vf[AHEAD];
            float m_new;
            int vis = n_vis;
            auto read_k = [&](int T, int i) { kf[i % AHEAD] = lds_ld16(kx[i] + T * K_TILE); };
            auto read_v = [&](int T, int i) {
              // registers 8s .. 8s+3 of the logits are keys 16s + 4kg + (0..3), registers 8s+4 .. 8s+7 the same + 8
              const uint32_t at = vx[i % NDT] + T * V_TILE + 16 * (i / NDT) * CH * 16;
              const uint2 lo = ds_read_tr16(at), hi = ds_read_tr16(at + 8 * CH * 16);
              vf[i % AHEAD] = make_uint4(lo.x, lo.y, hi.x, hi.y);
            };
            auto reference = [&]() {  // the row's maximum with the next tile
              float mx = nxt[0];
#pragma unroll
              for (int r = 1; r < 16; ++r) mx = fmaxf(mx, nxt[r]);
              mx = half_pair_max(mx);
              m_new = mx > NEG_BIG ? fmaxf(m_ref, fmaf(mx, p.scale2, HEADROOM)) : m_ref;
              m_sub = m_new > NEG_BIG ? m_new : 0.0f;
            };
            auto rescale = [&]() {
              if (__any(m_new > m_ref && l_sum > 0.0f)) {  // nothing to rescale before the first keys
                const float f = fast_exp2(m_ref - m_new);
                l_sum *= f;
#pragma unroll
                for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
                  for (int r = 0; r < 16; ++r) o[dt][r] *= f;
              }
              m_ref = m_new;
            };
            auto unit = [&](int T, bool more) {  // more: another tile follows
              uint4 pb[2];
              if (more)
#pragma unroll
                for (int r = 0; r < 16; ++r) nxt[r] = 0.0f;
#pragma unroll
              for (int i = 0; i < NCH; ++i) {
                if (more) Mma<DT>::run(nxt, kf[i % AHEAD], a[i]);
#pragma unroll
                for (int r = i * (16 / NCH); r < (i + 1) * (16 / NCH); ++r) {
                  x[r] = fast_exp2(x[r]);
                  l_sum += x[r];
                }
                if (i + AHEAD >= NCH) read_v(T, i + AHEAD - NCH);
                else if (more) read_k(T + 1, i + AHEAD);
                if (i == HALF - 1 || i == NCH - 1) {
                  const int s = i / HALF;
                  pb[s] = make_uint4(pack_bf16(x[8 * s], x[8 * s + 1]), pack_bf16(x[8 * s + 2], x[8 * s + 3]),
                                     pack_bf16(x[8 * s + 4], x[8 * s + 5]), pack_bf16(x[8 * s + 6], x[8 * s + 7]));
                }
                __builtin_amdgcn_sched_barrier(0);
              }
              if (more && !whole) hide(nxt, vis - (T + 1) * 32);
#pragma unroll
              for (int i = 0; i < NCH; ++i) {
                Mma<DT>::run(o[i % NDT], vf[i % AHEAD], pb[i / NDT]);
                if (i + AHEAD < NCH) read_v(T, i + AHEAD);
                else if (more) read_k(T + 2, i + AHEAD - NCH);
                if (more && i == HALF - 1) reference();
                if (more && i >= HALF)
#pragma unroll
                  for (int r = (i - HALF) * (16 / HALF); r < (i - HALF + 1) * (16 / HALF); ++r) x[r] = fmaf(nxt[r], p.scale2, -m_sub);
                __builtin_amdgcn_sched_barrier(0);
              }
              if (more) rescale();
            };
            if (left > 0) {
#pragma unroll
              for (int r = 0; r < 16; ++r) nxt[r] = 0.0f;
#pragma unroll
              for (int i = 0; i < AHEAD; ++i) read_k(0, i);
#pragma unroll
              for (int i = 0; i < NCH; ++i) {
                Mma<DT>::run(nxt, kf[i % AHEAD], a[i]);
                if (i + AHEAD < NCH) read_k(0, i + AHEAD);
                else read_k(1, i + AHEAD - NCH);
                __builtin_amdgcn_sched_barrier(0);
              }
              if (!whole) hide(nxt, vis);
              reference();
#pragma unroll
              for (int r = 0; r < 16; ++r) x[r] = fmaf(nxt[r], p.scale2, -m_sub);
              rescale();
              unit(0, true);
              for (; left > 2; left -= 2) {
                unit(1, true);
#pragma unroll
                for (int i = 0; i < NCH; ++i) kx[i] = opaque(kx[i] + 2 * K_TILE);
#pragma unroll
                for (int dt = 0; dt < NDT; ++dt) vx[dt] = opaque(vx[dt] + 2 * V_TILE);
                moved += 2 * K_TILE;
                vis -= 64;
                unit(0, true);
              }
              unit(1, false);
            }
          }
        } else {
          uint32_t kr = k_at + cur * (STAGE * 16) + nt0 * K_TILE, vr = v_at + cur * (STAGE * 16) + nt0 * V_TILE;
          int vis = n_vis;
#pragma unroll 1
          for (; left > 0; --left) {
            f32x16 acc;
            uint4 kf[NCH], vf[RUNS * NDT];
            load_k(kr, kf);
            logits(kf, acc);
            if (!whole) hide(acc, vis);
            soft(acc);
            load_v(vr, vf);
            weigh(acc, vf);
            kr += K_TILE;
            vr += V_TILE;
            vis -= 32;
          }
        }
        next();
        if (DT == DT_BF16) {
          const uint32_t move = (cur ? STAGE * 16 : -STAGE * 16) - moved;
#pragma unroll
          for (int i = 0; i < NCH; ++i) kx[i] = opaque(kx[i] + move);
#pragma unroll
          for (int dt = 0; dt < NDT; ++dt) vx[dt] = opaque(vx[dt] + move);
        }
      }
    }
    if (pass) {
      lds_barrier();  // every wave has left the stages
      break;
    }
    // once more (decided for the workgroup: the pass has barriers)
    if (bad || !finite()) *redo = 1;
    __syncthreads();
    if (!*redo) break;
    start(lo0);
    joined = single && have;
    nt0 = joined && !upper ? TPC / 2 : 0;
    load_rows(upper || single ? t_hi : t_lo);
    if (have) {
      land(0);
      lds_barrier();
    }
    while (have) {
      if (nhave) prefetch(nseg, nkc, cur ^ 1);
      if (!joined && seg && kc0 >= end_lo) {
        joined = true;
        if (!upper) load_rows(t_hi);
        nt0 = upper ? 0 : TPC / 2;
      }
      const int wave_end = seg ? min(hi1, upper || joined ? end_hi : end_lo) : hi0;
      int left = present ? min(min(max((wave_end - kc0 + 31) >> 5, 0), TPC) - nt0, joined ? TPC / 2 : TPC) : 0;
      const int lane_end = seg ? min(hi1, blk_end_lane) : hi0;
      for (int nt = nt0; left > 0; --left, ++nt) {
        const float mx = maximum(k_at + cur * (STAGE * 16) + nt * K_TILE, lane_end - (kc0 + nt * 32));
        float& ref = joined && !upper && !single ? ref_join : ref_own;
        ref = fmaxf(ref, mx);
      }
      next();
    }
    lds_barrier();
  }
  settle();
  // every wave has left the stages: the states of pairs that shared a tile meet there (rows padded by four floats
  // against bank conflicts)
  constexpr int OP = D + 4;
  static_assert((size_t)4 * 32 * (OP + 2) * 4 <= (size_t)2 * STAGE * 16, "the states do not fit the stages");
  const int tid_s = late(), kg_s = tid_s >> 5 & 1;
  float* so = reinterpret_cast<float*>(smem) + (size_t)((tid_s >> 6 & 3) * 32 + (tid_s & 31)) * OP;
  float2* sml = reinterpret_cast<float2*>(reinterpret_cast<float*>(smem) + (size_t)4 * 32 * OP) + (tid_s & 255);
  if (joined && !upper) {
#pragma unroll
    for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4)
        *reinterpret_cast<float4*>(so + dt * 32 + 8 * q4 + 4 * kg_s) =
            make_float4(o[dt][4 * q4], o[dt][4 * q4 + 1], o[dt][4 * q4 + 2], o[dt][4 * q4 + 3]);
    *sml = make_float2(m_ref, l_sum);
  }
  lds_barrier();
  if (!present) return;
  if (joined && upper) {
    const float2 ml = *sml;
    const float mn = fmaxf(m_ref, ml.x), wa = fast_exp2(m_ref - mn), wb = fast_exp2(ml.x - mn);
    m_ref = mn;
    l_sum = l_sum * wa + ml.y * wb;
#pragma unroll
    for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) {
        const float4 ov = *reinterpret_cast<const float4*>(so + dt * 32 + 8 * q4 + 4 * kg_s);
        const float of[4] = {ov.x, ov.y, ov.z, ov.w};
#pragma unroll
        for (int u = 0; u < 4; ++u) o[dt][4 * q4 + u] = o[dt][4 * q4 + u] * wa + of[u] * wb;
      }
  }
  if (upper) write_tile(t_hi);
  else if (!joined && !single) write_tile(t_lo);
}

// out = sum_p O_p 2^(m_p - M) / sum_p l_p 2^(m_p - M), lse = (M + log2 of that sum) ln 2.  A row takes D / 4 lanes across
// the head dimension times S slices of its partials, each slice merged on the fly and the slices then through LDS; a
// workgroup takes 8 / S rows, S growing with the partials (two partials of 24 000 rows with eight slices: 15 - 18 us,
// six of the slices idle; with two 9 us).  Without any partial (empty cache) the output is zero, the normaliser -inf.
constexpr int COMB_SLICES = 8;
template <int D, int S>
__global__ __launch_bounds__((D / 4) * COMB_SLICES) void attend_combine_kernel(AttendParams p) {
  constexpr int LPR = D / 4;  // lanes per row
  constexpr int ROWS = COMB_SLICES / S;
  __shared__ float4 sAcc[COMB_SLICES][LPR];
  __shared__ float2 sMl[COMB_SLICES];
  const int d4 = threadIdx.x % LPR, sl = threadIdx.x / LPR % S, rw = threadIdx.x / (LPR * S);
  // rows per split in the workspace, this row's first partial, and the row of the output (none: -1)
  int pitch = p.m_rows, row_lin = blockIdx.x * ROWS + rw;
  size_t first = 0;
  if (p.n_cut) {  // attend_rows_kernel's layout
    const int cut_wg = row_lin / ATT_ROWS, r = row_lin % ATT_ROWS, wg = p.n_full + cut_wg;
    const int h = wg / p.n_qgroups, pr = (wg - h * p.n_qgroups) * 4 + r / 64, n_tiles = (p.m_rows + 31) >> 5;
    const int t = r & 32 ? n_tiles - 1 - pr : pr, m = t * 32 + (r & 31);
    const bool none = pr >= (n_tiles + 1) / 2 || ((r & 32) && t == pr) || m >= p.m_rows;
    pitch = ATT_ROWS;
    row_lin = none ? -1 : h * p.m_rows + m;
    first = (size_t)cut_wg * p.n_parts * ATT_ROWS + r;
  } else if (row_lin < p.n_kv_heads * p.m_rows) {
    const int h = row_lin / p.m_rows;
    first = (size_t)h * p.n_parts * p.m_rows + (row_lin - h * p.m_rows);
  } else {
    row_lin = -1;
  }
  const float2* ml = p.part_ml + first;
  const float* po = p.part_o + first * D + d4 * 4;
  float mx = NEG_BIG, l = 0.0f;
  float4 acc = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
  if (row_lin >= 0) {
#pragma unroll 4
    for (int q = sl; q < p.n_parts; q += S) {
      const float2 v = ml[(size_t)q * pitch];
      const float4 ov = *reinterpret_cast<const float4*>(po + (size_t)q * pitch * D);
      const float mn = fmaxf(mx, v.x);
      const float wa = fast_exp2(mx - mn), wb = fast_exp2(v.x - mn);
      l = l * wa + v.y * wb;
      acc.x = acc.x * wa + ov.x * wb;
      acc.y = acc.y * wa + ov.y * wb;
      acc.z = acc.z * wa + ov.z * wb;
      acc.w = acc.w * wa + ov.w * wb;
      mx = mn;
    }
  }
  sAcc[rw * S + sl][d4] = acc;
  if (d4 == 0) sMl[rw * S + sl] = make_float2(mx, l);
  __syncthreads();
  if (sl != 0 || row_lin < 0) return;
  float mt = NEG_BIG;
#pragma unroll
  for (int k = 0; k < S; ++k) mt = fmaxf(mt, sMl[rw * S + k].x);
  float lt = 0.0f;
  float4 at = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
#pragma unroll
  for (int k = 0; k < S; ++k) {
    const float wgt = fast_exp2(sMl[rw * S + k].x - mt);
    const float4 ov = sAcc[rw * S + k][d4];
    lt = fmaf(sMl[rw * S + k].y, wgt, lt);
    at.x = fmaf(ov.x, wgt, at.x);
    at.y = fmaf(ov.y, wgt, at.y);
    at.z = fmaf(ov.z, wgt, at.z);
    at.w = fmaf(ov.w, wgt, at.w);
  }
  const float inv = lt > 0.0f ? 1.0f / lt : 0.0f;
  *reinterpret_cast<float4*>(p.out + (size_t)row_lin * D + d4 * 4) = make_float4(at.x * inv, at.y * inv, at.z * inv, at.w * inv);
  if (d4 == 0) p.out_lse[row_lin] = lt > 0.0f ? lse_log2(mt, lt) * 0.6931471805599453f : -__builtin_inff();
}

// ---------------------------------------------------------------------------------------------
// The normaliser alone (out == null): log sum_i exp(q.k_i / sqrt(d)) of every query over the cache, which is
// all laserkv_set_row_lse needs.  No values are read and no output accumulators kept, so a workgroup takes up to 512
// rows (a GQA group's whole window reads the keys once; with fewer rows the eight waves share them over different key
// tiles).  Workgroup = (key split, group of 512 rows, KV head); the arithmetic is laserkv_rowstats.h.
// 256 rows over 31 681 keys, 8 heads: 25.4-27 us, 27.7 a call with the merge in a series of calls (31.2 before products and
// exponentials were interleaved, 37 with sixteen waves of 32 rows, half of them without rows).
// ---------------------------------------------------------------------------------------------
constexpr int LSE_ROWS = 512;

template <int DT, int D, int RT, bool LONG>
__global__ __launch_bounds__(RS_THREADS) void attend_lse_kernel(AttendParams p) {
  constexpr int NCH = D * (DT == DT_BF16 ? 2 : 4) / 32;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, rl = lane & 31, kg = lane >> 5;
  const int idx = xcd_major(blockIdx.x, gridDim.x);
  const int split = idx % p.n_splits, rg = idx / p.n_splits % p.n_qgroups, h = idx / (p.n_splits * p.n_qgroups);
  const int k_lo = split * p.keys_per_split, k_hi = min(k_lo + p.keys_per_split, p.cache_len);
  const int wk = RS_WAVES >> p.wprt_log, wi = wave & ((1 << p.wprt_log) - 1), ks = wave >> p.wprt_log;
  const int row0 = rg * LSE_ROWS + wi * RT * 32;
  const bool active = row0 < p.m_rows;

  extern __shared__ uint4 smem[];
  uint4 q[RT][NCH];
  int lim[RT];
#pragma unroll
  for (int r = 0; r < RT; ++r) {
    const int m = min(row0 + r * 32 + rl, p.m_rows - 1);
    const int g = div_w(m, p.nq_magic), j = m - g * p.n_q;
    const char* ptr = p.q.base + (int64_t)(h * p.group + g) * p.q.stride_head + (int64_t)j * p.q.stride_row;
    lim[r] = k_hi;
#pragma unroll
    for (int i = 0; i < NCH; ++i) q[r][i] = ld16(ptr + (2 * i + kg) * 16);
  }
  const srd_words ksrd = make_srd_words(p.k_cache + (int64_t)h * p.cache_stride_head, (uint32_t)p.cache_len * (uint32_t)p.row_bytes);
  float ref[RT], sum[RT];
  row_stats<DT, D, RT, LONG>(smem, ksrd, (uint32_t)p.row_bytes, k_lo, k_hi, k_hi, lim, q, p.scale2, ks, wk, active, ref, sum);
  // the waves that shared rows meet in LDS (free after row_stats)
  float2* sP = reinterpret_cast<float2*>(smem);  // [wk][rows of the group]
  const int n_rows = RT * 32 << p.wprt_log;
#pragma unroll
  for (int r = 0; r < RT; ++r)
    if (kg == 0) sP[ks * n_rows + wi * RT * 32 + r * 32 + rl] = make_float2(ref[r], sum[r]);
  __syncthreads();
  const int row = rg * LSE_ROWS + tid;
  if (tid >= n_rows || row >= p.m_rows) return;
  float2 v = sP[tid];
  for (int k = 1; k < wk; ++k) lse_merge(v.x, v.y, sP[k * n_rows + tid].x, sP[k * n_rows + tid].y);
  p.part_ml[((size_t)h * p.n_parts + split) * p.m_rows + row] = v;
}

// lse = (M + log2 sum_p l_p 2^(m_p - M)) ln 2 per row; -inf without any partial (empty cache).  32 rows per workgroup,
// eight threads per row over the partials (one pass, their loads in flight together: 4.6 -> 2.5 us at 32 splits).
constexpr int LSEC_ROWS = 32, LSEC_SLICES = 8;
__global__ __launch_bounds__(LSEC_ROWS * LSEC_SLICES) void attend_lse_combine_kernel(AttendParams p) {
  __shared__ float2 sP[LSEC_SLICES][LSEC_ROWS];
  const int r = threadIdx.x % LSEC_ROWS, sl = threadIdx.x / LSEC_ROWS;
  const int row_lin = blockIdx.x * LSEC_ROWS + r, n_rows = p.n_kv_heads * p.m_rows;
  const int rc = min(row_lin, n_rows - 1);
  const int h = rc / p.m_rows, m = rc - h * p.m_rows;
  const float2* ml = p.part_ml + (size_t)h * p.n_parts * p.m_rows + m;
  float mx = NEG_BIG, l = 0.0f;
  for (int q0 = sl; q0 < p.n_parts; q0 += 8 * LSEC_SLICES) {
    float2 v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = ml[(size_t)min(q0 + u * LSEC_SLICES, p.n_parts - 1) * p.m_rows];
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (q0 + u * LSEC_SLICES < p.n_parts) lse_merge(mx, l, v[u].x, v[u].y);
  }
  sP[sl][r] = make_float2(mx, l);
  __syncthreads();
  if (sl || row_lin >= n_rows) return;
#pragma unroll
  for (int s = 1; s < LSEC_SLICES; ++s) lse_merge(mx, l, sP[s][r].x, sP[s][r].y);
  p.out_lse[row_lin] = l > 0.0f ? lse_log2(mx, l) * 0.6931471805599453f : -__builtin_inff();
}

// ---- host side ----
// Key splits for n_wg workgroups of attend_rows_kernel (one per compute unit at a time) that take t keys each.  The time is
// a line in t for every number of splits: rounds * (t keys / splits + a start), and with more than one the partials' way
// through memory and the merging launch.  The slopes fall as the splits that pay grow, so the choice grows with t and with
// it the workspace.
static int rows_splits(int n_wg, int n_cu, double t, int dtype, int head_dim) {
  const double key_us = 0.038 * head_dim / 128 * (dtype == DT_F32 ? 7.4 : 1.0);  // 256 rows; 0.030 over long ranges, 0.05 over 400 keys
  int best = 1;
  double best_cost = 0.0;
  for (int s = 1; s <= ATT_MAX_SPLITS; ++s) {
    const int rounds = (int)(((int64_t)n_wg * s + n_cu - 1) / n_cu);
    const double part_us = (double)n_wg * ATT_ROWS * head_dim * 8.0 / 6.0e6;  // a partial of every row written and read
    const double cost = rounds * (t / s * key_us + 4.0) + (s > 1 ? 4.0 + s * part_us : 0.0);
    if (s == 1 || cost < best_cost) {
      best = s;
      best_cost = cost;
    }
  }
  return best;
}

void attend_plan(int dtype, int head_dim, int m_rows, int n_q, int64_t cache_len, int s_t, int n_kv_heads, int n_cu, AttendPlan* plan) {
  if (decode_supports(m_rows, cache_len, s_t)) return decode_plan(cache_len, n_kv_heads, n_cu, plan);
  plan->decode = 0;
  const int n_rt = (m_rows + 31) / 32;
  if (n_rt > 4) {
    // a pair of waves per pair of row tiles.  The queries of a whole block see half of its keys on average
    const int n_pg = ((n_rt + 1) / 2 + 3) / 4;
    const double t = (double)cache_len + (2 * n_q > s_t ? 0.5 : 1.0) * s_t;
    // whole rounds of workgroups take all their keys; the workgroups of the last, incomplete round are cut by keys
    const int n_wg = n_kv_heads * n_pg, n_rest = n_wg % n_cu;
    const int s = n_rest ? min(rows_splits(n_rest, n_cu, t, dtype, head_dim), max(1, (int)((t + 31.0) / 32.0))) : 1;
    plan->n_qgroups = n_pg;
    plan->wprt_log = 0;
    plan->keys_per_split = plan->blk_keys_per_split = 0;  // the kernel cuts the ranges itself
    plan->n_cut = s > 1 ? n_rest : 0;
    plan->n_full = n_wg - plan->n_cut;
    plan->n_splits = plan->n_parts = s;
    return;
  }
  int rt_pow2 = 1, wprt_log = 3;
  while (rt_pow2 < n_rt) { rt_pow2 <<= 1; --wprt_log; }
  int n_splits = n_cu / n_kv_heads;
  n_splits = max(1, min(n_splits, ATT_MAX_SPLITS));
  // every split takes a share of the cache rows and a share of the block's keys
  int64_t kps = (cache_len + n_splits - 1) / n_splits;
  kps = max((int64_t)32, (kps + 31) / 32 * 32);
  int bps = (s_t + n_splits - 1) / n_splits;
  bps = max(32, (bps + 31) / 32 * 32);
  const int need_c = (int)((cache_len + kps - 1) / kps), need_b = (s_t + bps - 1) / bps;
  n_splits = max(need_c, need_b);  // 0: no key at all
  plan->n_qgroups = 1;
  plan->wprt_log = wprt_log;
  plan->n_splits = n_splits;
  plan->keys_per_split = (int)kps;
  plan->blk_keys_per_split = bps;
  plan->n_parts = n_splits;
  plan->n_full = plan->n_cut = 0;
}

void attend_lse_plan(int m_rows, int64_t cache_len, int n_kv_heads, int n_cu, AttendPlan* plan) {
  const int n_rg = (m_rows + LSE_ROWS - 1) / LSE_ROWS;
  int n_splits = n_cu / (n_kv_heads * n_rg);
  n_splits = max(1, min(n_splits, ATT_MAX_SPLITS));
  int64_t kps = (cache_len + n_splits - 1) / n_splits;
  kps = max((int64_t)32, (kps + 31) / 32 * 32);
  n_splits = cache_len > 0 ? (int)((cache_len + kps - 1) / kps) : 0;
  plan->n_qgroups = n_rg;
  // waves over different rows: two row tiles each (one where there are at most four); the others take other key tiles
  const int n_rt = (min(m_rows, LSE_ROWS) + 31) / 32, need = n_rt > 4 ? (n_rt + 1) / 2 : n_rt;
  plan->wprt_log = 0;
  while ((1 << plan->wprt_log) < need) ++plan->wprt_log;
  plan->n_splits = n_splits;
  plan->keys_per_split = (int)kps;
  plan->blk_keys_per_split = 32;
  plan->n_parts = n_splits;
  plan->n_full = plan->n_cut = plan->decode = 0;
}

size_t attend_part_rows(const AttendPlan& plan, int m_rows, int n_kv_heads) {
  if (plan.decode) return (size_t)n_kv_heads * plan.n_parts * decode_rows(m_rows);
  if (plan.n_full + plan.n_cut) return (size_t)plan.n_cut * plan.n_parts * ATT_ROWS;  // attend_rows_kernel
  return (size_t)n_kv_heads * plan.n_parts * m_rows;
}

size_t attend_workspace_bytes(const AttendPlan& plan, int m_rows, int n_kv_heads, int head_dim) {
  const size_t rows = attend_part_rows(plan, m_rows, n_kv_heads);
  return ((rows * head_dim * 4 + 255) & ~(size_t)255) + rows * 8 + 256;
}

template <int DT, int D, int KC>
static hipError_t launch_attend_kc(const AttendParams& p, hipStream_t st) {
  constexpr int ES = DT == DT_BF16 ? 2 : 4;
  constexpr size_t lds_chunk = ((size_t)KC * (D * ES / 16 + 1) + (size_t)D * (KC / (16 / ES) + 1)) * 16;
  constexpr size_t lds_merge = (size_t)ATT_WAVES * 32 * ((D + 4) * 4 + 8);  // the waves' states when they share row tiles
  constexpr size_t lds = lds_chunk > lds_merge ? lds_chunk : lds_merge;
  static_assert(lds <= 160 * 1024, "attention chunk does not fit the LDS");
  hipLaunchKernelGGL((attend_kernel<DT, D, KC>), dim3(p.n_splits * p.n_qgroups * p.n_kv_heads), dim3(ATT_THREADS), lds, st, p);
  return hipGetLastError();
}

template <int DT, int D>
static hipError_t launch_attend_t(const AttendParams& p, hipStream_t st) {
  if (p.n_full + p.n_cut) {
    constexpr int ES = DT == DT_BF16 ? 2 : 4;
    constexpr int KC = rows_chunk_keys<DT>();
    constexpr size_t v_stage = DT == DT_BF16 ? (size_t)KC * (D * ES / 16) : (size_t)D * (KC / (16 / ES) + 1);
    constexpr size_t lds = (size_t)2 * ((size_t)KC * (D * ES / 16) + v_stage) * 16 + 16;  // two stages and the redo flag
    static_assert(lds <= 160 * 1024, "two attention chunks do not fit the LDS");
    // The ring takes registers and a longer start.  Where no range is long enough for it, the instance without it: 50 rows
    // over 74 and 2691 keys 11.9 -> 11.7 and 21.5 -> 21.3 us, a block of 1298 rows without a cache 71.1 -> 70.3.  Without block
    // keys it pays from the shortest ranges on (256 rows, 384 a range: 35.3 -> 33.5 us).  Before a block, cut ranges run
    // over cache and block keys together, and the last ones, with the block's keys, decide: unless these hold many cache rows
    // too, the others only wait for them (eight heads, block of 2048 behind 6000 rows, 1760 a range and 720 in the last: 87.5
    // us without the ring, 89.4 with; 1024 rows of 32 heads behind 1500: 61.2, 62.7).
    const dim3 grid(p.n_full + p.n_cut * p.n_splits);
    const int n_tiles = (p.m_rows + 31) >> 5;
    bool ring = DT == DT_BF16 && p.cache_len > (p.s_t ? RING_KEYS : FIXED_KEYS);
    if (n_tiles <= 7 && (n_tiles & 1)) ring = false;  // the only workgroup of a range holds the tile that two waves share
    if (ring && !p.n_full) {
      const RowsShape shape = rows_shape(p);
      if (!p.s_t) ring = rows_cut(shape, 0, p.n_splits).share > FIXED_KEYS;
      else
        for (int pg = 0; pg < p.n_qgroups && ring; ++pg) ring = rows_last_cache_range(shape, pg, p.n_splits) > 2 * RING_KEYS;
    }
    if (DT == DT_BF16 && ring) hipLaunchKernelGGL((attend_rows_kernel<DT, D, DT == DT_BF16>), grid, dim3(ATT_THREADS), lds, st, p);
    else hipLaunchKernelGGL((attend_rows_kernel<DT, D, false>), grid, dim3(ATT_THREADS), lds, st, p);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess || !p.n_cut) return e;
  } else if (p.n_splits > 0) {
    const hipError_t e = launch_attend_kc<DT, D, att_chunk_keys<DT>()>(p, st);
    if (e != hipSuccess) return e;
  }
  const int n_rows = p.n_cut ? p.n_cut * ATT_ROWS : p.n_kv_heads * p.m_rows;
  const dim3 blk((D / 4) * COMB_SLICES);
  if (p.n_parts <= 3) hipLaunchKernelGGL((attend_combine_kernel<D, 2>), dim3((n_rows + 3) / 4), blk, 0, st, p);
  else if (p.n_parts <= 7) hipLaunchKernelGGL((attend_combine_kernel<D, 4>), dim3((n_rows + 1) / 2), blk, 0, st, p);
  else hipLaunchKernelGGL((attend_combine_kernel<D, 8>), dim3(n_rows), blk, 0, st, p);
  return hipGetLastError();
}

template <int DT, int D>
static hipError_t launch_attend_lse_t(const AttendParams& p, hipStream_t st) {
  if (p.n_splits > 0) {
    const dim3 grid(p.n_splits * p.n_qgroups * p.n_kv_heads), blk(RS_THREADS);
    const size_t lds = row_stats_lds(D * (DT == DT_BF16 ? 2 : 4));
    const int rt = min(p.m_rows, LSE_ROWS) > 128 ? 2 : 1;
    const bool lng = row_stats_long(DT, D * (DT == DT_BF16 ? 2 : 4), rt, p.keys_per_split);
    if (rt == 2 && lng) hipLaunchKernelGGL((attend_lse_kernel<DT, D, 2, DT == DT_BF16>), grid, blk, lds, st, p);
    else if (rt == 2) hipLaunchKernelGGL((attend_lse_kernel<DT, D, 2, false>), grid, blk, lds, st, p);
    else hipLaunchKernelGGL((attend_lse_kernel<DT, D, 1, false>), grid, blk, lds, st, p);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  const int n_rows = p.n_kv_heads * p.m_rows;
  hipLaunchKernelGGL(attend_lse_combine_kernel, dim3((n_rows + LSEC_ROWS - 1) / LSEC_ROWS), dim3(LSEC_ROWS * LSEC_SLICES), 0, st, p);
  return hipGetLastError();
}

hipError_t launch_attend_lse(int dtype, int head_dim, const AttendParams& p, hipStream_t st) {
  if (dtype == DT_BF16 && head_dim == 128) return launch_attend_lse_t<DT_BF16, 128>(p, st);
  if (dtype == DT_BF16 && head_dim == 64) return launch_attend_lse_t<DT_BF16, 64>(p, st);
  if (dtype == DT_F32 && head_dim == 128) return launch_attend_lse_t<DT_F32, 128>(p, st);
  if (dtype == DT_F32 && head_dim == 64) return launch_attend_lse_t<DT_F32, 64>(p, st);
  return hipErrorInvalidValue;
}

hipError_t launch_attend(int dtype, int head_dim, const AttendParams& p, hipStream_t st) {
  if (dtype == DT_BF16 && head_dim == 128) return launch_attend_t<DT_BF16, 128>(p, st);
  if (dtype == DT_BF16 && head_dim == 64) return launch_attend_t<DT_BF16, 64>(p, st);
  if (dtype == DT_F32 && head_dim == 128) return launch_attend_t<DT_F32, 128>(p, st);
  if (dtype == DT_F32 && head_dim == 64) return launch_attend_t<DT_F32, 64>(p, st);
  return hipErrorInvalidValue;
}

template <int DT, int D>
static hipError_t attend_attr() {
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&attend_kernel<DT, D, att_chunk_keys<DT>()>), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
  if (e == hipSuccess)
    e = hipFuncSetAttribute(reinterpret_cast<const void*>(&attend_rows_kernel<DT, D, false>), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
  if (e == hipSuccess)
    e = hipFuncSetAttribute(reinterpret_cast<const void*>(&attend_rows_kernel<DT, D, DT == DT_BF16>), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
  if (e == hipSuccess)
    e = hipFuncSetAttribute(reinterpret_cast<const void*>(&attend_lse_kernel<DT, D, 1, false>), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
  if (e == hipSuccess)
    e = hipFuncSetAttribute(reinterpret_cast<const void*>(&attend_lse_kernel<DT, D, 2, false>), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
  if (e == hipSuccess)
    e = hipFuncSetAttribute(reinterpret_cast<const void*>(&attend_lse_kernel<DT, D, 2, DT == DT_BF16>), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
  return e;
}

// Of the instances that a context can launch (each attribute takes some 4 us, and all types' were set for each)
hipError_t init_attend_attributes(int dtype, int head_dim) {
  if (dtype == DT_BF16) return head_dim == 128 ? attend_attr<DT_BF16, 128>() : attend_attr<DT_BF16, 64>();
  return head_dim == 128 ? attend_attr<DT_F32, 128>() : attend_attr<DT_F32, 64>();
}

}  // namespace lkv

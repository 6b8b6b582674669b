// Attention of very few query rows per KV head over the compacted cache (a decoding step: G * n_q <= 8 rows).
//
// Reading K and V once bounds this (one query per head over 63 520 rows: 260 MB), and the arithmetic is small enough
// for the vector unit, so nothing passes through LDS on the way: a row of K or V is 16 bytes per lane across
// D * elem size / 16 consecutive lanes, loaded whole, coalesced and streaming.  A logit is a partial dot product per
// lane and a DPP reduction over the row's lanes; each of them ends with the logit of ONE query row (l % M), takes one
// exponential, and the rows' probabilities spread through quad broadcasts to the lanes, which hold the same key's piece
// of V: the weighted sum is in-lane.  Each group of lanes keeps its own online-softmax state over its keys; groups,
// waves and key splits are merged at the end, the splits by the last workgroup of a head to finish: one launch, whose
// 4 us of counter and loads on the memory side cost the GPU what a second kernel did and the host 2.6 us less.
//
// Workgroup = (key split, KV head), 8 waves that never wait for each other in the main loop.  K of the next tile is
// requested as soon as the current tile's logits are done and V as soon as its sum is done.
//
// Measured (32/8 heads, d 128, bf16, one query): 7301 rows 13.3 -> 11.5 us (of which 1.8 launch, 8 until the keys are
// worked off, 4 merging), 63 520 rows 52.4 -> 43.4 us = 6.0 TB/s (loads alone: 40 us).  The matrix-instruction kernel
// before it passed everything through LDS with a register transpose of V and two barriers per 256 keys.
#include "laserkv_device.h"
#include "laserkv_kernels.h"

namespace lkv {

constexpr int DEC_WAVES = 8;
constexpr int DEC_MAX_SPLITS = 64;  // a wave's lanes hold a row's splits

// K and V are read once: streaming loads leave the caches to other data and run at 6.9 instead of 6.0 TB/s
__device__ __forceinline__ uint4 buf_ld16_stream(__amdgpu_buffer_rsrc_t r, uint32_t byte_offset) {
  const u32x4_ld v = __builtin_amdgcn_raw_buffer_load_b128(r, (int)byte_offset, 0, 2);
  return make_uint4(v.x, v.y, v.z, v.w);
}

template <int CTRL>
__device__ __forceinline__ float dpp_mov(float v) {
  return __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(v), CTRL, 0xf, 0xf, true));
}
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_mov(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xf, 0xf, true);
}
constexpr int DPP_XOR1 = 0xB1, DPP_XOR2 = 0x4E, DPP_ROR4 = 0x124, DPP_ROR8 = 0x128;

// M values per lane, each to be summed over the N lanes of a row: halving the values with every exchange, lane l ends
// with the sum of value l % M (8 steps for four values over sixteen lanes instead of 16).
template <int M, int N>
__device__ __forceinline__ float row_sums(const float* s, int lane) {
  const bool b0 = lane & 1, b1 = lane & 2, b2 = lane & 4;
  float t[M];
#pragma unroll
  for (int m = 0; m < M; ++m) t[m] = s[m];
  int done = 1;  // lanes summed over so far
  if (M >= 2) {
#pragma unroll
    for (int m = 0; m < M / 2; ++m) t[m] = (b0 ? t[2 * m + 1] : t[2 * m]) + dpp_mov<DPP_XOR1>(b0 ? t[2 * m] : t[2 * m + 1]);
    done = 2;
  }
  if (M >= 4) {
#pragma unroll
    for (int m = 0; m < M / 4; ++m) t[m] = (b1 ? t[2 * m + 1] : t[2 * m]) + dpp_mov<DPP_XOR2>(b1 ? t[2 * m] : t[2 * m + 1]);
    done = 4;
  }
  if (M >= 8) {
    t[0] = (b2 ? t[1] : t[0]) + __uint_as_float(lane_xor4(__float_as_uint(b2 ? t[0] : t[1]), b2));
    done = 8;
  }
  float v = t[0];
  if (done < 2) v += dpp_mov<DPP_XOR1>(v);
  if (done < 4) v += dpp_mov<DPP_XOR2>(v);
  if (N == 8) {
    if (done < 8) v += __uint_as_float(lane_xor4(__float_as_uint(v), b2));
  } else {
    if (done < 8) v += dpp_mov<DPP_ROR4>(v);
    v += dpp_mov<DPP_ROR8>(v);
  }
  if (N == 32) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  }
  return v;
}
// the value of lane m of the quad (M <= 4) in all its lanes
template <typename T>
__device__ __forceinline__ T quad_of(T v, int m) {
  switch (m) {
    case 0: return dpp_mov<0x00>(v);
    case 1: return dpp_mov<0x55>(v);
    case 2: return dpp_mov<0xAA>(v);
    default: return dpp_mov<0xFF>(v);
  }
}
// lane l holds the value of query row l % M: every lane gets those of all M rows
template <int M, typename T>
__device__ __forceinline__ void rows_all(T v, int lane, T* out) {
  if (M == 1) {
    out[0] = v;
  } else if (M <= 4) {
#pragma unroll
    for (int m = 0; m < M; ++m) out[m] = quad_of(v, m);
  } else {
    const bool b2 = lane & 4;
    const T other = __builtin_bit_cast(T, lane_xor4(__builtin_bit_cast(uint32_t, v), b2));
    const T lo = b2 ? other : v, hi = b2 ? v : other;
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      out[m] = quad_of(lo, m);
      out[4 + m] = quad_of(hi, m);
    }
  }
}
// maximum over the lanes l, l ^ N, ... that hold the same piece of different rows (N lanes per row)
template <int N>
__device__ __forceinline__ float groups_max(float v) {
  if (N <= 8) v = fmaxf(v, dpp_mov<DPP_ROR8>(v));
  if (N <= 16) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
  }
  return half_pair_max(v);
}
template <int N>
__device__ __forceinline__ float groups_sum(float v) {
  if (N <= 8) v += dpp_mov<DPP_ROR8>(v);
  if (N <= 16) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  }
  return half_pair_sum(v);
}

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ float dot2(uint32_t a, uint32_t b, float c) {
  return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, a), __builtin_bit_cast(bf16x2, b), c, false);
}
// partial dot product of two 16-byte pieces
template <int DT>
__device__ __forceinline__ float dot16(const uint4& a, const uint4& b) {
  if (DT == DT_BF16) return dot2(a.w, b.w, dot2(a.z, b.z, dot2(a.y, b.y, dot2(a.x, b.x, 0.0f))));
  float s = __uint_as_float(a.x) * __uint_as_float(b.x);
  s = fmaf(__uint_as_float(a.y), __uint_as_float(b.y), s);
  s = fmaf(__uint_as_float(a.z), __uint_as_float(b.z), s);
  return fmaf(__uint_as_float(a.w), __uint_as_float(b.w), s);
}

// Partials travel between workgroups (possibly on different XCDs) as device-scope relaxed stores and loads, which are
// served at the memory side; the order is "stores acknowledged, then the counter" and "counter seen, then the loads".
__device__ __forceinline__ void dec_store(uint64_t* p, float a, float b) {
  __hip_atomic_store(p, (uint64_t)__float_as_uint(a) | ((uint64_t)__float_as_uint(b) << 32), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float2 dec_load(const uint64_t* p) {
  const uint64_t v = __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return make_float2(__uint_as_float((uint32_t)v), __uint_as_float((uint32_t)(v >> 32)));
}

// M: query rows the kernel keeps (>= p.m_rows).
template <int DT, int D, int M>
__global__ __launch_bounds__(DEC_WAVES * 64) void attend_decode_kernel(AttendParams p) {
  constexpr int ES = DT == DT_BF16 ? 2 : 4;
  constexpr int LPK = D * ES / 16;   // lanes per row
  constexpr int KPL = 64 / LPK;      // rows per load
  constexpr int EPC = 16 / ES;       // elements per lane
  constexpr int U = 4;               // loads per tile and tensor
  constexpr int TK = U * KPL;        // keys per tile
  constexpr int DEC_THREADS = DEC_WAVES * 64;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int idx = xcd_major(blockIdx.x, gridDim.x);
  const int h = idx / p.n_splits, split = idx - h * p.n_splits;
  const int lo = min(split * p.keys_per_split, p.cache_len), hi = min(lo + p.keys_per_split, p.cache_len);
  const int c = lane % LPK, sub = lane / LPK;

  constexpr int PAIRS = M * D / 2;               // a thread per pair of outputs
  constexpr int GRP = DEC_THREADS / PAIRS;       // groups of threads in the last merge
  static_assert(PAIRS <= DEC_THREADS && GRP * PAIRS == DEC_THREADS, "threads divide into whole groups");
  constexpr int LANES = GRP > DEC_WAVES ? GRP : DEC_WAVES;
  __shared__ float sO[LANES][M][D];
  __shared__ float2 sML[DEC_WAVES][M];     // the waves' (reference, sum)
  __shared__ float sW[DEC_MAX_SPLITS][M];  // the splits' weights
  __shared__ float2 sTotal[M];
  __shared__ int sLast;

  uint4 q[M];
#pragma unroll
  for (int m = 0; m < M; ++m) {
    const int mc = min(m, p.m_rows - 1), g = div_w(mc, p.nq_magic), j = mc - g * p.n_q;
    q[m] = ld16(p.q.base + (int64_t)(h * p.group + g) * p.q.stride_head + (int64_t)j * p.q.stride_row + c * 16);
  }
  const uint32_t rb = (uint32_t)p.row_bytes;
  const __amdgpu_buffer_rsrc_t ksrd = make_srd(p.k_cache + (int64_t)h * p.cache_stride_head, (uint32_t)p.cache_len * rb);
  const __amdgpu_buffer_rsrc_t vsrd = make_srd(p.v_cache + (int64_t)h * p.cache_stride_head, (uint32_t)p.cache_len * rb);
  uint4 k[U], v[U];
  auto load = [&](uint4* r, __amdgpu_buffer_rsrc_t srd, int key0) {  // rows past the cache read as zero
    const uint32_t at = (uint32_t)(key0 + sub) * rb + c * 16;
#pragma unroll
    for (int u = 0; u < U; ++u) r[u] = buf_ld16_stream(srd, at + u * KPL * rb);
  };

  // lane l keeps reference and sum of query row l % M over its group's keys; the weighted sums of all rows at the
  // lane's piece of the head dimension
  float ref = NEG_BIG, sum = 0.0f, o[M * EPC];
#pragma unroll
  for (int e = 0; e < M * EPC; ++e) o[e] = 0.0f;
  int t0 = lo + wave * TK;
  if (t0 < hi) {
    load(k, ksrd, t0);
    load(v, vsrd, t0);
  }
#pragma unroll 1
  for (; t0 < hi; t0 += DEC_WAVES * TK) {
    const int next = t0 + DEC_WAVES * TK;
    float s[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      float part[M];
#pragma unroll
      for (int m = 0; m < M; ++m) part[m] = dot16<DT>(k[u], q[m]);
      s[u] = row_sums<M, LPK>(part, lane);
    }
    if (next < hi) load(k, ksrd, next);
    if (t0 + TK > hi) {  // wave-uniform: the split's last tile
#pragma unroll
      for (int u = 0; u < U; ++u) s[u] = t0 + u * KPL + sub < hi ? s[u] : -__builtin_inff();
    }
    float mx = s[0];
#pragma unroll
    for (int u = 1; u < U; ++u) mx = fmaxf(mx, s[u]);
    mx *= p.scale2;  // scale2 > 0
    // the reference follows the maximum: the largest probability is exactly 1, also as the bf16 that weighs V, so a row
    // that one key dominates gets that key's values unrounded (raised only past 2^8 it was off by up to 2^-9 of them)
    if (__any(mx > ref)) {
      const float nref = fmaxf(ref, mx), f = fast_exp2(ref - nref);
      sum *= f;
      float fm[M];
      rows_all<M>(f, lane, fm);
#pragma unroll
      for (int m = 0; m < M; ++m)
#pragma unroll
        for (int e = 0; e < EPC; ++e) o[m * EPC + e] *= fm[m];
      ref = nref;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      s[u] = fast_exp2(fmaf(s[u], p.scale2, -ref));
      sum += s[u];
    }
    if (DT == DT_BF16) {
      // two keys at a time: their values as pairs, their probabilities rounded to bf16 (as the matrix path does)
#pragma unroll
      for (int u = 0; u < U; u += 2) {
        bf16x2 pp = {(__bf16)s[u], (__bf16)s[u + 1]};
        uint32_t pm[M];
        rows_all<M>(__builtin_bit_cast(uint32_t, pp), lane, pm);
        const uint32_t a[4] = {v[u].x, v[u].y, v[u].z, v[u].w}, b[4] = {v[u + 1].x, v[u + 1].y, v[u + 1].z, v[u + 1].w};
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          const uint32_t even = __builtin_amdgcn_perm(b[w], a[w], 0x05040100u), odd = __builtin_amdgcn_perm(b[w], a[w], 0x07060302u);
#pragma unroll
          for (int m = 0; m < M; ++m) {
            o[m * EPC + 2 * w % EPC] = dot2(even, pm[m], o[m * EPC + 2 * w % EPC]);
            o[m * EPC + (2 * w + 1) % EPC] = dot2(odd, pm[m], o[m * EPC + (2 * w + 1) % EPC]);
          }
        }
      }
    } else {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        float pm[M];
        rows_all<M>(s[u], lane, pm);
        const uint32_t a[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
#pragma unroll
        for (int w = 0; w < 4; ++w)
#pragma unroll
          for (int m = 0; m < M; ++m) o[m * EPC + w % EPC] = fmaf(pm[m], __uint_as_float(a[w]), o[m * EPC + w % EPC]);
      }
    }
    if (next < hi) load(v, vsrd, next);
  }

  // the wave's groups of lanes: one reference, the sums halved with every exchange, so that a lane ends with
  // M * EPC * LPK / 64 outputs
  {
    const float mx = groups_max<LPK>(ref), f = fast_exp2(ref - mx);
    sum = groups_sum<LPK>(sum * f);
    float fm[M];
    rows_all<M>(f, lane, fm);
#pragma unroll
    for (int m = 0; m < M; ++m)
#pragma unroll
      for (int e = 0; e < EPC; ++e) o[m * EPC + e] *= fm[m];
    constexpr int N0 = M * EPC, N1 = N0 / 2, N2 = LPK <= 16 ? N1 / 2 : N1, N3 = LPK <= 8 ? N2 / 2 : N2;
    int at = (lane >> 5) * N1;  // first output of this lane, as row * EPC + element
#pragma unroll
    for (int i = 0; i < N1; ++i) {
      const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(o[i]), __float_as_uint(o[i + N1]), false, false);
      o[i] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    }
    if (LPK <= 16) {
      at += ((lane >> 4) & 1) * N2;
#pragma unroll
      for (int i = 0; i < N2; ++i) {
        const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(o[i]), __float_as_uint(o[i + N2]), false, false);
        o[i] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
      }
    }
    if (LPK <= 8) {
      const bool up = lane & 8;
      at += up ? N3 : 0;
#pragma unroll
      for (int i = 0; i < N3; ++i) o[i] = (up ? o[i + N3] : o[i]) + dpp_mov<DPP_ROR8>(up ? o[i] : o[i + N3]);
    }
#pragma unroll
    for (int i = 0; i < N3; ++i) sO[wave][(at + i) / EPC][c * EPC + (at + i) % EPC] = o[i];
    if (lane < M) sML[wave][lane] = make_float2(mx, sum);
  }
  __syncthreads();
  const size_t rows0 = (size_t)h * p.m_rows;
  uint64_t* part = reinterpret_cast<uint64_t*>(p.part_o);   // [H_kv, n_splits, M, D / 2] pairs
  uint64_t* part_ml = reinterpret_cast<uint64_t*>(p.part_ml);  // [H_kv, n_splits, M]
  const int m = tid / (D / 2), d2 = tid % (D / 2);
  const bool own = tid < PAIRS && m < p.m_rows;
  float l = 0.0f, mx = NEG_BIG;
  float2 acc = make_float2(0.0f, 0.0f);
  if (own) {
#pragma unroll
    for (int w = 0; w < DEC_WAVES; ++w) mx = fmaxf(mx, sML[w][m].x);
#pragma unroll
    for (int w = 0; w < DEC_WAVES; ++w) {
      const float2 ml = sML[w][m];
      const float f = fast_exp2(ml.x - mx);
      const float2 ov = *reinterpret_cast<const float2*>(&sO[w][m][2 * d2]);
      l = fmaf(ml.y, f, l);
      acc.x = fmaf(ov.x, f, acc.x);
      acc.y = fmaf(ov.y, f, acc.y);
    }
  }
  if (p.n_splits > 1) {
    const size_t at = ((size_t)h * p.n_splits + split) * M + m;
    if (own) {
      dec_store(part + at * (D / 2) + d2, acc.x, acc.y);
      if (d2 == 0) dec_store(part_ml + at, mx, l);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this wave's partials are acknowledged
    __syncthreads();
    if (tid == 0) sLast = __hip_atomic_fetch_add(p.counters + h, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (uint32_t)p.n_splits - 1u;
    __syncthreads();
    if (!sLast) return;
    if (tid == 0) __hip_atomic_store(p.counters + h, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);  // for the next launch
    // every thread takes a pair of outputs of every GRP-th split, NOV at a time, all requested before the first use;
    // wave m turns row m's references into weights meanwhile (lane = split)
    constexpr int NOV = GRP > 2 ? 8 : 16;
    const int grp = tid / PAIRS, pm = tid % PAIRS / (D / 2);
    const uint64_t* po = part + ((size_t)h * p.n_splits * M + min(pm, p.m_rows - 1)) * (D / 2) + d2;
    float2 ov[NOV];
    auto fetch = [&](int i0) {
#pragma unroll
      for (int u = 0; u < NOV; ++u) ov[u] = dec_load(po + (size_t)min(i0 + u * GRP, p.n_splits - 1) * M * (D / 2));
    };
    if (wave < p.m_rows) {
      float2 ml = make_float2(NEG_BIG, 0.0f);
      if (lane < p.n_splits) ml = dec_load(part_ml + ((size_t)h * p.n_splits + lane) * M + wave);
      fetch(grp);
      float wm = ml.x;
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) wm = fmaxf(wm, __shfl_xor(wm, off));
      const float f = fast_exp2(ml.x - wm);
      float wl = ml.y * f;
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) wl += __shfl_xor(wl, off);
      sW[lane][wave] = f;
      if (lane == 0) sTotal[wave] = make_float2(wm, wl);
    } else {
      fetch(grp);
    }
    __syncthreads();
    acc = make_float2(0.0f, 0.0f);
    for (int i0 = grp; i0 < p.n_splits; i0 += NOV * GRP) {
      if (i0 != grp) fetch(i0);
#pragma unroll
      for (int u = 0; u < NOV; ++u) {
        const float f = i0 + u * GRP < p.n_splits ? sW[i0 + u * GRP][min(pm, p.m_rows - 1)] : 0.0f;
        acc.x = fmaf(ov[u].x, f, acc.x);
        acc.y = fmaf(ov[u].y, f, acc.y);
      }
    }
    if (own) {
      mx = sTotal[m].x;
      l = sTotal[m].y;
    }
    if (GRP > 1) {  // the groups' sums meet in LDS, where the waves' were
      *reinterpret_cast<float2*>(&sO[grp][pm][2 * d2]) = acc;
      __syncthreads();
      if (!own) return;
      acc = *reinterpret_cast<const float2*>(&sO[0][m][2 * d2]);
#pragma unroll
      for (int g = 1; g < GRP; ++g) {
        const float2 og = *reinterpret_cast<const float2*>(&sO[g][m][2 * d2]);
        acc.x += og.x;
        acc.y += og.y;
      }
    }
  }
  if (!own) return;
  const float inv = l > 0.0f ? 1.0f / l : 0.0f;  // all logits -inf (products that overflow): zero and -inf
  *reinterpret_cast<float2*>(p.out + (rows0 + m) * D + 2 * d2) = make_float2(acc.x * inv, acc.y * inv);
  if (d2 == 0) p.out_lse[rows0 + m] = l > 0.0f ? (mx + fast_log2(l)) * 0.6931471805599453f : -__builtin_inff();
}

// ---- host side ----
// Up to eight rows the vector unit keeps up with the memory (about a third of its rate at four rows, two thirds at
// eight); more go to attend_kernel's matrix instructions.
bool decode_supports(int m_rows, int64_t cache_len, int s_t) { return m_rows <= 8 && s_t == 0 && cache_len > 0; }

void decode_plan(int64_t cache_len, int n_kv_heads, int n_cu, AttendPlan* plan) {
  // a workgroup per compute unit; at least a tile of 32 keys for every second wave, so that short caches are not cut
  // into more partials than they have work
  int n_splits = n_cu / n_kv_heads;
  n_splits = n_splits < 1 ? 1 : (n_splits > DEC_MAX_SPLITS ? DEC_MAX_SPLITS : n_splits);
  int64_t kps = (cache_len + n_splits - 1) / n_splits;
  kps = kps < 128 ? 128 : (kps + 31) / 32 * 32;
  n_splits = (int)((cache_len + kps - 1) / kps);
  plan->n_qgroups = 1;
  plan->wprt_log = 0;
  plan->n_splits = n_splits;
  plan->keys_per_split = (int)kps;
  plan->blk_keys_per_split = 32;
  plan->n_parts = n_splits;
  plan->n_full = plan->n_cut = 0;
  plan->decode = 1;
}

template <int DT, int D>
static hipError_t launch_decode_t(const AttendParams& p, hipStream_t st) {
  // eight waves with four loads per tensor in flight; sixteen waves, eight loads or two workgroups per compute unit
  // measure the same or slower (11.6 - 14.3 us and 46.6 - 48.4 us on the two contexts below)
  const dim3 grid(p.n_splits * p.n_kv_heads), blk(DEC_WAVES * 64);
  if (p.m_rows <= 1) hipLaunchKernelGGL((attend_decode_kernel<DT, D, 1>), grid, blk, 0, st, p);
  else if (p.m_rows <= 2) hipLaunchKernelGGL((attend_decode_kernel<DT, D, 2>), grid, blk, 0, st, p);
  else if (p.m_rows <= 4) hipLaunchKernelGGL((attend_decode_kernel<DT, D, 4>), grid, blk, 0, st, p);
  else hipLaunchKernelGGL((attend_decode_kernel<DT, D, 8>), grid, blk, 0, st, p);
  return hipGetLastError();
}

hipError_t launch_decode(int dtype, int head_dim, const AttendParams& p, hipStream_t st) {
  if (dtype == DT_BF16 && head_dim == 128) return launch_decode_t<DT_BF16, 128>(p, st);
  if (dtype == DT_BF16 && head_dim == 64) return launch_decode_t<DT_BF16, 64>(p, st);
  if (dtype == DT_F32 && head_dim == 128) return launch_decode_t<DT_F32, 128>(p, st);
  if (dtype == DT_F32 && head_dim == 64) return launch_decode_t<DT_F32, 64>(p, st);
  return hipErrorInvalidValue;
}
int decode_rows(int m_rows) { return m_rows <= 2 ? m_rows : (m_rows <= 4 ? 4 : 8); }

}  // namespace lkv

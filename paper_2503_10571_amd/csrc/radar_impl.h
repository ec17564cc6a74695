// Internal declarations shared by the translation units of libradar.so:
// the device helpers every kernel uses (sequence spans, element conversion,
// streaming loads, DPP exchanges, the top-k and union building blocks, the
// attention tile), the host-side shape and workspace types, the launch
// helper, and the launchers each unit provides to the others. Not part of
// the C ABI (include/radar.h is).
#pragma once

#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <type_traits>
#include <vector>

#include "radar.h"

namespace radar_impl {

constexpr float kLog2e = 1.44269504088896340736f;
constexpr int kWave = 64;
constexpr int kTile = 64;          // tokens per attention tile and per key tile of k_build_f32
constexpr int kMaxK = 256;         // largest k accepted
constexpr int kMaxG = 8;           // largest query-head group
constexpr int kMaxCand = 2048;     // largest number of candidate segments
constexpr int kMaxWg = 1024;       // largest attention split per (b, kv head)
constexpr int kFusedMaxCand = 1024;   // candidates whose scores fit in LDS

typedef uint16_t bf16_t;           // storage type of a bfloat16 value
typedef unsigned long long u64;   // 64-bit type of the wave shuffles
typedef __attribute__((__vector_size__(8 * sizeof(short)))) short bf16x8_t;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4_t;
typedef __bf16 bf16x2v_t __attribute__((ext_vector_type(2)));

// ---------------------------------------------------------------------------
// token layout of one sequence at a decode step
// ---------------------------------------------------------------------------
// A sequence of length len starts with sink = min(n_sink, len) attention-sink
// tokens. The kernels address K / V from the first row after the sinks
// (the host offsets the pointers by n_sink rows), so in these row numbers
// candidate segment s covers [s c, s c + c) for s < n_cand, the window is
// [ws, t) with t = len - sink and ws = c floor(max(0, t - w) / c), and the
// sinks are rows [-n_sink, -n_sink + sink). A length outside [1, t_max]
// marks the sequence invalid: it selects nothing, attends nothing, and its
// outputs are NaN.
struct SeqArgs {
  const int64_t* lens;  // [B] per-sequence lengths (device), or null: all t_max
  int64_t t_max;
  int c, w, n_sink, k;
  int lens_add = 0;     // 1: lens holds append rows, a sequence's length is
                        // its row + 1 (0, invalid, unless row < t_max)
};

// Lengths stay below 2^31 (the capacity limit), so the split is computed in
// 32-bit arithmetic.
struct Span {
  int t, ws, n_cand, k_eff, sink;
  bool ok;
};

__host__ __device__ inline Span make_span(int64_t len, const SeqArgs& a) {
  Span p;
  p.ok = len >= 1 && len <= a.t_max;
  const int L = p.ok ? (int)len : 0;
  p.sink = L < a.n_sink ? L : a.n_sink;
  p.t = L - p.sink;
  const unsigned past = p.t > a.w ? (unsigned)(p.t - a.w) : 0u;
  p.n_cand = (int)(past / (unsigned)a.c);
  p.ws = p.n_cand * a.c;
  p.k_eff = p.n_cand < a.k ? p.n_cand : a.k;
  return p;
}

__device__ __forceinline__ Span seq_span(const SeqArgs& a, int64_t b) {
  if (!a.lens) return make_span(a.t_max, a);
  const int64_t v = a.lens[b];
  if (!a.lens_add) return make_span(v, a);
  return make_span(v >= 0 && v < a.t_max ? v + 1 : 0, a);
}

// The k / v row write of an append. radar_append runs it as its own kernel;
// radar_append_decode runs it inside the per-(b, kv head) kernel that
// precedes every read of the row, one wave per pair.
struct AppendArgs {
  uint4* K;                // cache base (row 0 of pair 0); null: no append
  uint4* V;
  const uint4* kn;         // [B][Hkv] rows of the new keys / values
  const uint4* vn;
  const int64_t* pos;      // [B] row of sequence b, or null: row t for all
  int64_t t;
  int chunks;              // 16-byte chunks per row
};

// rows outside [0, cap) are skipped
__device__ __forceinline__ void append_row(const AppendArgs& ap, int64_t cap,
                                           int64_t bh, int Hkv, int lane) {
  const int64_t row = ap.pos ? ap.pos[bh / Hkv] : ap.t;
  if (row < 0 || row >= cap) return;
  const int64_t dst = (bh * cap + row) * ap.chunks, src = bh * ap.chunks;
  for (int i = lane; i < ap.chunks; i += kWave) {
    ap.K[dst + i] = ap.kn[src + i];
    ap.V[dst + i] = ap.vn[src + i];
  }
}

// union entries: segment id in the low 16 bits, the mask of the group's
// query heads that selected it in bits 16 .. 23
constexpr int kUniIdBits = 16;
constexpr unsigned kAllHeads = 0xffu;

// ---------------------------------------------------------------------------
// element helpers
// ---------------------------------------------------------------------------
template <typename T> struct Elem;
template <> struct Elem<float> { static constexpr int kPer16 = 4; };
template <> struct Elem<bf16_t> { static constexpr int kPer16 = 8; };

__device__ __forceinline__ float bf16_lo(uint32_t x) {
  return __uint_as_float(x << 16);
}
__device__ __forceinline__ float bf16_hi(uint32_t x) {
  return __uint_as_float(x & 0xffff0000u);
}

// 16 bytes -> floats
template <typename T>
__device__ __forceinline__ void unpack16(const uint4& u, float* f);
template <>
__device__ __forceinline__ void unpack16<float>(const uint4& u, float* f) {
  f[0] = __uint_as_float(u.x); f[1] = __uint_as_float(u.y);
  f[2] = __uint_as_float(u.z); f[3] = __uint_as_float(u.w);
}
template <>
__device__ __forceinline__ void unpack16<bf16_t>(const uint4& u, float* f) {
  f[0] = bf16_lo(u.x); f[1] = bf16_hi(u.x);
  f[2] = bf16_lo(u.y); f[3] = bf16_hi(u.y);
  f[4] = bf16_lo(u.z); f[5] = bf16_hi(u.z);
  f[6] = bf16_lo(u.w); f[7] = bf16_hi(u.w);
}

// fp32 -> bf16, round to nearest even; infinities stay infinite and NaN
// becomes a quiet NaN (a select, not a branch)
__device__ __forceinline__ uint32_t f32_to_bf16(float f) {
  const uint32_t u = __float_as_uint(f);
  const uint32_t rounded = (u + 0x7fffu + ((u >> 16) & 1u)) >> 16;
  const uint32_t qnan = (u >> 16) | 0x40u;
  return (u & 0x7fffffffu) > 0x7f800000u ? qnan : rounded;
}
__device__ __forceinline__ float round_bf16(float f) {
  return __uint_as_float(f32_to_bf16(f) << 16);
}

template <typename T> __device__ __forceinline__ T from_f32(float f);
template <> __device__ __forceinline__ float from_f32<float>(float f) { return f; }
template <> __device__ __forceinline__ bf16_t from_f32<bf16_t>(float f) {
  return (bf16_t)f32_to_bf16(f);
}
template <typename T> __device__ __forceinline__ float to_f32(T v);
template <> __device__ __forceinline__ float to_f32<float>(float v) { return v; }
template <> __device__ __forceinline__ float to_f32<bf16_t>(bf16_t v) {
  return __uint_as_float(((uint32_t)v) << 16);
}

__device__ __forceinline__ float fast_exp2(float x) {
  return __builtin_amdgcn_exp2f(x);
}

// Non-temporal 16-byte loads for data read once per launch (K/V tiles, key
// tiles, summary rows): they stream past the caches and sustain a higher
// HBM read rate than ordinary loads on MI355X.
typedef unsigned u32x4_t __attribute__((ext_vector_type(4)));
typedef float f32x4v_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint4 ld_stream(const void* p) {
  const u32x4_t t = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(p));
  return make_uint4(t.x, t.y, t.z, t.w);
}
__device__ __forceinline__ float4 ld_stream_f4(const float* p) {
  const f32x4v_t t = __builtin_nontemporal_load(reinterpret_cast<const f32x4v_t*>(p));
  return make_float4(t.x, t.y, t.z, t.w);
}

// ---------------------------------------------------------------------------
// cross-lane exchanges
// ---------------------------------------------------------------------------
// DPP controls (GFX9): quad_perm [1,0,3,2] and [2,3,0,1] swap neighbours at
// distance 1 and 2; row_half_mirror maps lane i of each 8-lane half-row to
// 7 - i, row_mirror maps lane i of each 16-lane row to 15 - i;
// row_newbcast:n copies lane n of every row to the whole row.
constexpr int kDppQuadSwap1 = 0xB1;
constexpr int kDppQuadSwap2 = 0x4E;
constexpr int kDppHalfMirror = 0x141;
constexpr int kDppMirror = 0x140;
constexpr int kDppRowBcast0 = 0x150;
constexpr int kDppRowRor0 = 0x120;         // + n: lane i of a row takes lane i - n mod 16

// the value of lane l ^ MASK of the 16-lane row, for any MASK below 16
template <int MASK>
__device__ __forceinline__ float row_xor(float v) {
  static_assert(MASK == 1 || MASK == 2 || MASK == 4 || MASK == 8, "distance");
  const int x = __float_as_int(v);
  if constexpr (MASK == 1) return __int_as_float(__builtin_amdgcn_mov_dpp(x, kDppQuadSwap1, 0xf, 0xf, true));
  else if constexpr (MASK == 2) return __int_as_float(__builtin_amdgcn_mov_dpp(x, kDppQuadSwap2, 0xf, 0xf, true));
  else if constexpr (MASK == 8) return __int_as_float(__builtin_amdgcn_mov_dpp(x, kDppRowRor0 + 8, 0xf, 0xf, true));
  else {
    // quads 0 and 2 take the quad above (row_shl:4), 1 and 3 the one below
    const int up = __builtin_amdgcn_update_dpp(x, x, 0x104, 0xf, 0x5, false);
    return __int_as_float(__builtin_amdgcn_update_dpp(up, x, 0x114, 0xf, 0xa, false));
  }
}

// compile-time loop: f(std::integral_constant<int, I>) for I = B .. E-1
template <int B, int E, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (B < E) {
    f(std::integral_constant<int, B>{});
    static_for<B + 1, E>(f);
  }
}

// (a plain DPP move, every lane's source valid for these controls: the
// compiler folds it into the add or max that consumes it)
template <int CTRL>
__device__ __forceinline__ float dpp_f(float v) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xf, 0xf, true));
}

// Lanes l and l ^ 16 (MASK 16) or l and l ^ 32 (MASK 32) exchange on the
// vector ALUs: v_permlane16_swap / v_permlane32_swap with both operands the
// same value leave, in every lane, the pair's two values (the lower lane's
// first) in the two results.
template <int MASK>
__device__ __forceinline__ void xor_pair(float v, float& lo, float& hi) {
  static_assert(MASK == 16 || MASK == 32, "permlane swap distance");
  const unsigned u = __float_as_uint(v);
  if constexpr (MASK == 16) {
    const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    lo = __uint_as_float(r[0]); hi = __uint_as_float(r[1]);
  } else {
    const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    lo = __uint_as_float(r[0]); hi = __uint_as_float(r[1]);
  }
}
// v plus the value of lane l ^ MASK (MASK 16 or 32; the same sum in both
// lanes of the pair)
template <int MASK>
__device__ __forceinline__ float xor_sum(float v) {
  float lo, hi;
  xor_pair<MASK>(v, lo, hi);
  return lo + hi;
}

// Value of the partner lane in a pairing that differs from this lane in bit
// MASK. Within a 16-lane row the pairings are DPP moves (mirrors for bits 3
// and 2, quad swaps for bits 1 and 0); they are only used from the highest
// bit down, so the lower bits still to be processed never matter. Bits 4
// and 5 are lane l ^ MASK, by permlane swaps.
template <int MASK>
__device__ __forceinline__ float partner(float x, int lane) {
  if constexpr (MASK == 1) return dpp_f<kDppQuadSwap1>(x);
  else if constexpr (MASK == 2) return dpp_f<kDppQuadSwap2>(x);
  else if constexpr (MASK == 4) return dpp_f<kDppHalfMirror>(x);
  else if constexpr (MASK == 8) return dpp_f<kDppMirror>(x);
  else {
    float lo, hi;
    xor_pair<MASK>(x, lo, hi);
    return (lane & MASK) ? lo : hi;
  }
}

// One step of a cross-lane transpose-reduce: NV values per lane; paired lanes
// (different bit MASK) keep complementary halves, chosen by their own bit
// MASK, and add the partner's copy of the kept half.
template <int NV, int MASK>
__device__ __forceinline__ void halve(float* v, int lane) {
  const bool up = (lane & MASK) != 0;
#pragma unroll
  for (int i = 0; i < NV / 2; ++i) {
    const float keep = up ? v[i + NV / 2] : v[i];
    const float send = up ? v[i] : v[i + NV / 2];
    v[i] = keep + partner<MASK>(send, lane);
  }
}

// Reduce NV partial sums (one per row i) held by every lane of each group of
// NV consecutive lanes: afterwards lane j of the group holds row j's total.
template <int NV>
__device__ __forceinline__ void transpose_reduce(float* v, int lane) {
  if constexpr (NV >= 64) halve<64, 32>(v, lane);
  if constexpr (NV >= 32) halve<32, 16>(v, lane);
  if constexpr (NV >= 16) halve<16, 8>(v, lane);
  if constexpr (NV >= 8) halve<8, 4>(v, lane);
  if constexpr (NV >= 4) halve<4, 2>(v, lane);
  if constexpr (NV >= 2) halve<2, 1>(v, lane);
}

// 16-lane row all-reduce (every lane of a row ends with the row's result)
__device__ __forceinline__ float row_max(float v) {
  v = fmaxf(v, dpp_f<kDppQuadSwap1>(v));
  v = fmaxf(v, dpp_f<kDppQuadSwap2>(v));
  v = fmaxf(v, dpp_f<kDppHalfMirror>(v));
  return fmaxf(v, dpp_f<kDppMirror>(v));
}
__device__ __forceinline__ float row_sum(float v) {
  v += dpp_f<kDppQuadSwap1>(v);
  v += dpp_f<kDppQuadSwap2>(v);
  v += dpp_f<kDppHalfMirror>(v);
  return v + dpp_f<kDppMirror>(v);
}
__device__ __forceinline__ float lane_read(float v, int l) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}
// wave-wide results, uniform across the wave (rows combined by readlane)
__device__ __forceinline__ float wave_max(float v) {
  v = row_max(v);
  return fmaxf(fmaxf(lane_read(v, 0), lane_read(v, 16)),
               fmaxf(lane_read(v, 32), lane_read(v, 48)));
}
__device__ __forceinline__ float wave_sum(float v) {
  v = row_sum(v);
  return (lane_read(v, 0) + lane_read(v, 16)) + (lane_read(v, 32) + lane_read(v, 48));
}


// ---------------------------------------------------------------------------
// top-k helpers
// ---------------------------------------------------------------------------
// Order key of (score, index): larger key = better; ties in score go to the
// lower segment index. Keys are unique because indices are; 0 = no segment.
__device__ __forceinline__ u64 order_key(float s, int idx) {
  uint32_t u = __float_as_uint(s);
  u = (u & 0x80000000u) ? ~u : (u | 0x80000000u);
  return ((u64)u << 32) | (u64)(0xffffffffu - (uint32_t)idx);
}
__device__ __forceinline__ int key_index(u64 key) {
  return (int)(0xffffffffu - (uint32_t)(key & 0xffffffffu));
}
__device__ __forceinline__ float key_score(u64 key) {
  uint32_t u = (uint32_t)(key >> 32);
  u = (u & 0x80000000u) ? (u & 0x7fffffffu) : ~u;
  return __uint_as_float(u);
}

// Top-k_eff of one query head by one wave, k-independent. Lane l holds
// candidates m * 64 + l (m < NPL: coalesced loads). The k_eff-th largest
// 32-bit score key is found bit by bit, from the highest bit in which the
// present keys differ down (the bits above it are common to all of them): at
// each bit every lane counts its keys that match the prefix found so far and
// have the bit set, a DPP reduction sums the counts, and the bit is kept
// when at least the still-needed number of keys has it. The search stops
// once every key matching the prefix is needed. Then every key above the
// threshold and the lowest-index keys equal to it are compacted into LDS
// (positions from a prefix sum of per-lane counts; only when more keys tie
// at the threshold than are needed does the index order of the ties take
// one ballot per register) and rank-sorted by (score desc, index asc).
// list: k words of LDS owned by this wave. Vector counts and scans: no LDS
// atomics (candidates of similar scores share their leading bits, so a
// histogram over those bits sends every key to one bin) and no ballot per
// key and bit.
template <int CTRL>
__device__ __forceinline__ int dpp_i(int v) {
  return __builtin_amdgcn_mov_dpp(v, CTRL, 0xf, 0xf, true);
}
// AND / OR over the 64 lanes, uniform: the 16-lane row by DPP (quad swaps,
// mirrors), then the rows by permlane swaps
__device__ __forceinline__ uint32_t wave_and_u32(uint32_t v) {
  int x = (int)v;
  x &= dpp_i<kDppQuadSwap1>(x);
  x &= dpp_i<kDppQuadSwap2>(x);
  x &= dpp_i<kDppHalfMirror>(x);
  x &= dpp_i<kDppMirror>(x);
  float lo, hi;
  xor_pair<16>(__int_as_float(x), lo, hi);
  x = __float_as_int(lo) & __float_as_int(hi);
  xor_pair<32>(__int_as_float(x), lo, hi);
  x = __float_as_int(lo) & __float_as_int(hi);
  return (uint32_t)__builtin_amdgcn_readfirstlane(x);
}
__device__ __forceinline__ uint32_t wave_or_u32(uint32_t v) {
  int x = (int)v;
  x |= dpp_i<kDppQuadSwap1>(x);
  x |= dpp_i<kDppQuadSwap2>(x);
  x |= dpp_i<kDppHalfMirror>(x);
  x |= dpp_i<kDppMirror>(x);
  float lo, hi;
  xor_pair<16>(__int_as_float(x), lo, hi);
  x = __float_as_int(lo) | __float_as_int(hi);
  xor_pair<32>(__int_as_float(x), lo, hi);
  x = __float_as_int(lo) | __float_as_int(hi);
  return (uint32_t)__builtin_amdgcn_readfirstlane(x);
}
// sum over the 64 lanes, uniform
__device__ __forceinline__ int wave_sum_i32(int v) {
  v += dpp_i<kDppQuadSwap1>(v);
  v += dpp_i<kDppQuadSwap2>(v);
  v += dpp_i<kDppHalfMirror>(v);
  v += dpp_i<kDppMirror>(v);
  return (__builtin_amdgcn_readlane(v, 0) + __builtin_amdgcn_readlane(v, 16)) +
         (__builtin_amdgcn_readlane(v, 32) + __builtin_amdgcn_readlane(v, 48));
}
// inclusive prefix sum over the 64 lanes
__device__ __forceinline__ int wave_incl_scan(int v, int lane) {
  int x = v;
  x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);   // row_shr:1
  x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);   // row_shr:2
  x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);   // row_shr:4
  x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);   // row_shr:8
  const int r0 = __builtin_amdgcn_readlane(x, 15);
  const int r1 = __builtin_amdgcn_readlane(x, 31);
  const int r2 = __builtin_amdgcn_readlane(x, 47);
  const int row = lane >> 4;
  return x + (row > 0 ? r0 : 0) + (row > 1 ? r1 : 0) + (row > 2 ? r2 : 0);
}

template <int NPL>
__device__ void head_topk(const float* __restrict__ src, int n_cand, int k,
                          int k_eff, int* sel_row, int32_t* sel_out,
                          float* sc_out, int lane, u64* list) {
  uint32_t u[NPL];                         // ordered score keys, 0 = absent
  if (n_cand > 0) {
    float v[NPL];
#pragma unroll
    for (int m = 0; m < NPL; ++m) v[m] = src[min(m * 64 + lane, n_cand - 1)];
#pragma unroll
    for (int m = 0; m < NPL; ++m)
      u[m] = (m * 64 + lane < n_cand) ? (uint32_t)(order_key(v[m], 0) >> 32) : 0u;
  } else {
#pragma unroll
    for (int m = 0; m < NPL; ++m) u[m] = 0u;
  }
  if (k_eff > 0) {
    // bits common to every present key (absent keys count as neither)
    uint32_t kand = 0xffffffffu, kor = 0u;
#pragma unroll
    for (int m = 0; m < NPL; ++m)
      if (u[m] != 0u) { kand &= u[m]; kor |= u[m]; }
    kand = wave_and_u32(kand);
    kor = wave_or_u32(kor);
    const uint32_t diff = kand ^ kor;
    const int top = diff ? 31 - __clz((int)diff) : -1;
    // (prefix, mask): the leading bits of the k_eff-th largest key found so
    // far; `need` keys are still to take among those matching them (every
    // key with larger leading bits is taken)
    uint32_t mask = top >= 0 ? ~((2u << top) - 1u) : 0xffffffffu;
    uint32_t prefix = kand & mask;
    int need = k_eff;
#pragma unroll 1
    for (int bit = top; bit >= 0; --bit) {
      const uint32_t mb = mask | (1u << bit);
      const uint32_t pb = prefix | (1u << bit);
      int c = 0;
#pragma unroll
      for (int m = 0; m < NPL; ++m) c += ((u[m] & mb) == pb) ? 1 : 0;
      const int cnt = wave_sum_i32(c);
      mask = mb;
      if (cnt >= need) {
        prefix = pb;
        // every key left with these leading bits is taken
        if (cnt == need) break;
      } else {
        need -= cnt;
      }
    }
    // take every key whose leading bits are larger, and the `need`
    // lowest-index keys whose leading bits equal them
    int n_gt = 0, n_eq = 0;
#pragma unroll
    for (int m = 0; m < NPL; ++m) {
      const uint32_t um = u[m] & mask;
      n_gt += um > prefix ? 1 : 0;
      n_eq += (um == prefix && u[m] != 0u) ? 1 : 0;
    }
    const bool all_eq = wave_sum_i32(n_eq) == need;   // uniform
    // eq_take[m]: whether this lane's key m is a tie that is taken
    uint32_t eq_take = 0u;
    if (all_eq) {
#pragma unroll
      for (int m = 0; m < NPL; ++m)
        eq_take |= ((u[m] & mask) == prefix && u[m] != 0u) ? 1u << m : 0u;
    } else {
      // more ties than needed: the lowest indices, m * 64 + lane order
      const u64 lt_mask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
      int before = 0;
#pragma unroll
      for (int m = 0; m < NPL; ++m) {
        const bool eq = (u[m] & mask) == prefix && u[m] != 0u;
        const u64 be = __ballot(eq);
        if (eq && before + (int)__popcll(be & lt_mask) < need) eq_take |= 1u << m;
        before += __popcll(be);
      }
    }
    const int n_take = n_gt + __popc(eq_take);
    int pos = wave_incl_scan(n_take, lane) - n_take;
#pragma unroll
    for (int m = 0; m < NPL; ++m) {
      if ((u[m] & mask) > prefix || ((eq_take >> m) & 1u)) {
        list[pos] = ((u64)u[m] << 32) | (u64)(0xffffffffu - (uint32_t)(m * 64 + lane));
        ++pos;
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    // rank sort of the k_eff selected keys (larger key first)
    for (int i = lane; i < k_eff; i += 64) {
      const u64 key = list[i];
      int rank = 0;
#pragma unroll 8
      for (int j = 0; j < k_eff; ++j) rank += list[j] > key ? 1 : 0;
      const int idx = key_index(key);
      sel_row[rank] = idx;
      if (sel_out) sel_out[rank] = idx;
      if (sc_out) sc_out[rank] = key_score(key);
    }
  }
  for (int r = k_eff + lane; r < k; r += 64) {
    if (sel_out) sel_out[r] = -1;
    if (sc_out) sc_out[r] = __uint_as_float(0x7fc00000u);
  }
}

// A segment's score is the same bits on every path, whatever shares its batch:
// the n features are taken in chunks of 256 (all of them below that), lane l
// holding four consecutive ones (n / 64 below 256). A chunk's products are one
// fma chain per lane, then added over the 16 lanes of a row and over the four
// rows; the chunks are added pairwise, (0 + 1) + (2 + 3) and so on, so that any
// split of them into aligned runs (slices, waves) adds up to the same sum.
//
// tree_add takes the chunks' values one by one (at most eight) and returns the
// sum at the last.
__device__ __forceinline__ float tree_add(float v, int i, float (&hold)[3]) {
  if (i & 1) {
    v = hold[0] + v;
    if (i & 2) {
      v = hold[1] + v;
      if (i & 4) v = hold[2] + v;
      else hold[2] = v;
    } else {
      hold[1] = v;
    }
  } else {
    hold[0] = v;
  }
  return v;
}

// One head's scores from nsl (2, 4 or 8) slices of the features, `stride` floats
// apart, added pairwise into dst (LDS) by one wave, up to 32 loads in flight.
// Only where there are at most kFusedMaxCand candidates.
__device__ __forceinline__ void add_slices(const float* __restrict__ src, int nsl, int64_t stride,
                                           int n_cand, float* dst, int lane) {
  for (int i0 = 0; i0 < n_cand; i0 += 4 * kWave) {
    float x[8][4];
#pragma unroll
    for (int z = 0; z < 8; ++z)
#pragma unroll
      for (int m = 0; m < 4; ++m)
        x[z][m] = src[min(z, nsl - 1) * stride + min(i0 + m * kWave + lane, n_cand - 1)];
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      const float two = x[0][m] + x[1][m];
      const float four = two + (x[2][m] + x[3][m]);
      const float eight = four + ((x[4][m] + x[5][m]) + (x[6][m] + x[7][m]));
      const int i = i0 + m * kWave + lane;
      if (i < n_cand) dst[i] = nsl == 2 ? two : nsl == 4 ? four : eight;
    }
  }
  // (the wave reads what it wrote)
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Union of the group's selections: sel[h * per .. h * per + per) holds the
// segment ids of head h < G (-1 = none, every other id < kMaxCand). The ids
// are set in an LDS bitmap (one per head when masks are wanted); the first
// wave ORs the heads' words and turns the popcounts into prefix offsets, and
// then every thread of the workgroup lists some of the set bits: the
// distinct ids in ascending order go to uni, each with the mask of the heads
// that chose it (all heads without masks), and their count to *ucnt. bits:
// G * kMaxCand / 32 words of LDS. A barrier-synchronised call of the whole
// workgroup; the caller orders sel's writes before it and uni's reads after.
constexpr int kBitmapWords = kMaxCand / 32;
static_assert(kBitmapWords == kWave, "one bitmap word per lane");
__device__ inline void group_union(const int* sel, unsigned* bits, int G, int per,
                            bool masks, int* uni, int* ucnt) {
  // each word's union over the maps, and its exclusive prefix of set bits
  __shared__ uint32_t or_lds[kBitmapWords];
  __shared__ int pre_lds[kBitmapWords];
  const int tid = threadIdx.x;
  const int nmaps = masks ? G : 1;
  for (int i = tid; i < nmaps * kBitmapWords; i += blockDim.x) bits[i] = 0u;
  __syncthreads();
  for (int i = tid; i < G * per; i += blockDim.x) {
    const int id = sel[i];
    const int map = masks ? i / per : 0;
    if (id >= 0) atomicOr(&bits[map * kBitmapWords + (id >> 5)], 1u << (id & 31));
  }
  __syncthreads();
  if (tid < kWave) {
    uint32_t word = 0u;
    for (int g = 0; g < nmaps; ++g) word |= bits[g * kBitmapWords + tid];
    const int pc = __popc(word);
    // exclusive prefix sum of the popcounts over the 64 lanes
    int incl = pc;
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
      const int o = __shfl_up(incl, d);
      if (tid >= d) incl += o;
    }
    or_lds[tid] = word;
    pre_lds[tid] = incl - pc;
    if (tid == kWave - 1) *ucnt = incl;
  }
  __syncthreads();
  // every thread lists some of the set bits: id i sits at its word's
  // prefix plus the set bits below it in the word (ascending ids)
  for (int i = tid; i < kBitmapWords * 32; i += blockDim.x) {
    const int w = i >> 5, bit = i & 31;
    const uint32_t word = or_lds[w];
    if ((word >> bit) & 1u) {
      unsigned m = kAllHeads;
      if (masks) {
        m = 0u;
        for (int g = 0; g < nmaps; ++g) m |= ((bits[g * kBitmapWords + w] >> bit) & 1u) << g;
      }
      uni[pre_lds[w] + __popc(word & ((1u << bit) - 1u))] = i | (int)(m << kUniIdBits);
    }
  }
}

// ---------------------------------------------------------------------------
// exact attention over <= 64-token tiles (shared by k_attend and k_decode_fused)
// ---------------------------------------------------------------------------
// The attended tokens of a (b, kv head) are cut into tiles of <= 64 tokens
// that never cross a segment or the window boundary; a wave attends one tile
// after another with an online softmax (running max m and sum l in log2
// units, unreduced accumulators). TileMfma serves bf16 caches, TileVec fp32
// ones; run() walks a wave's tiles, finish() leaves its state in LDS.
struct TileRef {
  int64_t row0;     // first row of the tile, counted from the base pointers
  int len;          // 1 .. 64 rows
  unsigned hmask;   // head g of the group takes part only if bit g is set
};

// fp32 caches, on the vector ALUs: lane (r, jj) (r = lane / LPR) reads the
// 16-byte chunk jj of rows r, r + RPI, ... so every load instruction covers
// RPI whole rows contiguously (rows past the tile end re-read its last row
// and are masked). q.k partials (fma of the pre-scaled query) are
// transpose-reduced so that each lane ends with one token's logit, softmax
// runs across the wave, and p is broadcast back (DPP row broadcast) to the
// lanes that hold the matching V chunks. At d = 128 the 64 rows of K and V take
// 256 registers, which k_attend has for one or two heads (IT = 32: a step of 96
// pairs of 8.4 MB with two heads 112 us, 129 in halves; of 1.0 MB 32 and 40;
// with one head 137 and 154); with more heads, and in the 512-thread workgroups
// of the scored kernel, a tile is done in two halves of 32 rows (IT = 16: 75 us
// instead of 120 for 40 pairs of 3.3 MB with eight heads).
template <int D, int G, int IT = 16>
struct TileVec {
  static constexpr int kLdsBytes = 0;           // per wave
  static constexpr int EPL = 4;                 // elements per 16-byte chunk
  static constexpr int LPR = D / EPL;           // lanes per row: 16 or 32
  static constexpr int RPI = kWave / LPR;       // rows per load instruction
  static constexpr int ITER = IT;               // load instructions per pass
  static constexpr int ROWS = ITER * RPI;       // rows per pass: 64 or 32
  static_assert(ITER == 16 || ITER == LPR, "tile shape");

  float qf[G][EPL];
  float m[G], l[G], acc[G][EPL];
  int lane;

  // q0: the group's first query head; qscale folds log2(e) / sqrt(d)
  __device__ __forceinline__ void init(const float* __restrict__ q0, float qscale, int ln) {
    lane = ln;
    const int jj = lane % LPR;
#pragma unroll
    for (int g = 0; g < G; ++g) {
      unpack16<float>(*reinterpret_cast<const uint4*>(q0 + g * D + jj * EPL), qf[g]);
#pragma unroll
      for (int e = 0; e < EPL; ++e) { qf[g][e] *= qscale; acc[g][e] = 0.f; }
      m[g] = -INFINITY;
      l[g] = 0.f;
    }
  }

  // rows [row0, row0 + len), len <= ROWS (a head that has attended nothing
  // yet keeps m = -inf, l = 0, acc = 0)
  __device__ __forceinline__ void pass(const float* __restrict__ K, const float* __restrict__ V,
                                       int64_t row0, int len, unsigned hmask) {
    const int r = lane / LPR;
    const int jj = lane % LPR;
    uint4 kr[ITER], vr[ITER];
    const float* kbase = K + row0 * D + jj * EPL;
    const float* vbase = V + row0 * D + jj * EPL;
#pragma unroll
    for (int i = 0; i < ITER; ++i)
      kr[i] = ld_stream(kbase + (int64_t)min(i * RPI + r, len - 1) * D);
#pragma unroll
    for (int i = 0; i < ITER; ++i)
      vr[i] = ld_stream(vbase + (int64_t)min(i * RPI + r, len - 1) * D);

    // logits: lane (r, jj) ends with the logit of row (jj % ITER) * RPI + r
    // (in a half tile lanes jj and jj + 16 both hold it)
    float lg[G];
    {
      float pl[G][ITER];
#pragma unroll
      for (int i = 0; i < ITER; ++i) {
        float kf[EPL];
        unpack16<float>(kr[i], kf);
#pragma unroll
        for (int g = 0; g < G; ++g) {
          float a = 0.f;
#pragma unroll
          for (int e = 0; e < EPL; ++e) a = fmaf(qf[g][e], kf[e], a);
          pl[g][i] = a;
        }
      }
#pragma unroll
      for (int g = 0; g < G; ++g) {
        transpose_reduce<ITER>(pl[g], lane);
        lg[g] = LPR != ITER ? xor_sum<16>(pl[g][0]) : pl[g][0];
      }
    }
    const bool mine_ok = ((jj % ITER) * RPI + r) < len;
    float p[G];
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const bool on = mine_ok && ((hmask >> g) & 1u);
      const float mt = wave_max(on ? lg[g] : -INFINITY);
      const float mn = fmaxf(m[g], mt);
      const float mref = mn == -INFINITY ? 0.f : mn;
      const float scale = fast_exp2(m[g] - mref);  // 0 on the head's first tile
      p[g] = on ? fast_exp2(lg[g] - mref) : 0.f;
      l[g] = fmaf(l[g], scale, wave_sum(jj < ITER ? p[g] : 0.f));
      m[g] = mn;
#pragma unroll
      for (int e = 0; e < EPL; ++e) acc[g][e] *= scale;
    }
    static_for<0, ITER>([&](auto ic) {
      constexpr int i = decltype(ic)::value;
      float vf[EPL];
      unpack16<float>(vr[i], vf);
#pragma unroll
      for (int g = 0; g < G; ++g) {
        // p of row (i, r) lives in lane i of its row's lanes (of both 16-lane
        // rows of them in a half tile)
        float pb;
        if constexpr (ITER == 16) pb = dpp_f<kDppRowBcast0 + i>(p[g]);
        else pb = __shfl(p[g], r * LPR + i);
#pragma unroll
        for (int e = 0; e < EPL; ++e) acc[g][e] = fmaf(pb, vf[e], acc[g][e]);
      }
    });
  }
  __device__ __forceinline__ void tile(const float* K, const float* V, const TileRef& t) {
    if constexpr (ROWS == kTile) {
      pass(K, V, t.row0, t.len, t.hmask);
    } else {
#pragma unroll 1
      for (int off = 0; off < t.len; off += ROWS)
        pass(K, V, t.row0 + off, min(ROWS, t.len - off), t.hmask);
    }
  }

  // tiles first, first + step, ... < end of at(i); wave-uniform call
  template <typename At>
  __device__ __forceinline__ void run(const float* K, const float* V, int first, int end, int step,
                                      unsigned char*, At&& at) {
    for (int i = first; i < end; i += step) tile(K, V, at(i));
  }

  // the wave's totals: acc of head g, dim e to wacc[g * D + e], its maximum
  // and sum to wm[g] and wl[g]
  __device__ __forceinline__ void finish(float* wacc, float* wm, float* wl) {
    static_for<0, 6>([&](auto bc) {
      constexpr int msk = 1 << decltype(bc)::value;
      if constexpr (msk >= LPR) {
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
          for (int e = 0; e < EPL; ++e) {
            if constexpr (msk >= 16) acc[g][e] = xor_sum<msk>(acc[g][e]);
            else acc[g][e] += __shfl_xor(acc[g][e], msk);
          }
      }
    });
    if (lane < LPR) {
#pragma unroll
      for (int g = 0; g < G; ++g)
#pragma unroll
        for (int e = 0; e < EPL; ++e) wacc[g * D + lane * EPL + e] = acc[g][e];
    }
    if (lane == 0) {
#pragma unroll
      for (int g = 0; g < G; ++g) { wm[g] = m[g]; wl[g] = l[g]; }
    }
  }
};

// bf16 caches, on the matrix cores. Both products are 16x16x32 MFMAs whose 16
// columns are query heads, so their cost does not depend on the group:
//   S[token][head] = K Q^T    A = 16 keys, B = the group's queries
//   O^T[dim][head] += V^T P^T A = 16 dims, B = p of 32 tokens
// K goes from memory to the wave's own 16 KB (d = 128) of LDS by direct loads
// of whole rows, 16-byte chunk c of row x at place c ^ swz(x), which makes the
// A-operand reads free of bank conflicts. (Loading K straight into A-operand
// registers instead touches 16 cache lines per quarter wave: 5.9 against 6.9
// TB/s for whole rows, by registers or by LDS alike.) V goes to registers in
// whole rows too, lane (r, jj) holding chunk jj of tokens 4 i + r: for each
// element e of the chunk those are one row (dim EV jj + e) of V^T at the
// k-slots of lane group r, so two-register byte permutes make the operand
// and no value crosses lanes. The rows of S are assigned to tokens so that
// the logits a lane ends up with are exactly its k-slots of P^T: a lane's
// row 4 grp + j of sub-tile st is token 16 st + 4 j + grp.
//
// p stays exact: its 24 bits are cut into three bf16 terms (truncations, the
// last remainder is exact) and the unused columns take them. Up to four heads
// the 16 columns hold the head's term 0, 1 and 2 at col, col + G and
// col + 2 G and one product does all three; with eight heads the columns hold
// terms 0 and 1 and a second product adds term 2. The terms' sums are added
// at the end. A term is never 0 where p is not (an infinite V times a zero
// term would be NaN where p V is infinite).
//
// The next tile's K is requested as soon as the logits are out of LDS and its
// V as soon as this tile's V is used, so a wave has loads in flight while it
// computes.
//
// Against one dot2 and fma chain per head on the vector ALUs (the tile before
// this one, 1570 vector instructions at four heads and twice that at eight,
// with K in registers and nothing in flight during them): 167 against 183 us
// for 16 sequences of 64K tokens with four heads per group, 80 against 90 us
// at 512K, 104 against 211 us for six sequences of 32K with eight heads
// (485 MB); 109 us either way at 128K with one head, which streams at the
// read rate.
template <int D, int G>
struct TileMfma {
  static constexpr int KB = D / 32;             // MFMA steps of q.k
  static constexpr int EV = D / 16;             // V elements per lane and row
  static constexpr int CPR = D / 8;             // 16-byte chunks per row
  static constexpr int RPI = kWave / CPR;       // rows per K load
  static constexpr int NS = kTile / 16;         // 16-token sub-tiles
  static constexpr int NV = kTile / 4;          // V loads per tile
  static constexpr int kLdsBytes = kTile * D * 2;   // per wave
  static constexpr int kTerms = G <= 4 ? 3 : 2; // terms of p in the columns
  typedef typename std::conditional<EV == 8, uint4, uint2>::type VRow;

  bf16x8_t qb[KB];
  f32x4_t acc[EV];
  float m, l, qs;
  uint32_t cut0, cut1;      // masks that cut the lane's term out of p
  int lane;

  __device__ static __forceinline__ int swz(int row) {
    return D == 128 ? row & 15 : (row >> 1) & 7;
  }

  __device__ __forceinline__ void init(const bf16_t* __restrict__ q0, float qscale, int ln) {
    lane = ln;
    qs = qscale;
    const int col = lane & 15, grp = lane >> 4;
    const int term = col / G;
#pragma unroll
    for (int kb = 0; kb < KB; ++kb)
      qb[kb] = *reinterpret_cast<const bf16x8_t*>(q0 + (col % G) * D + kb * 32 + grp * 8);
#pragma unroll
    for (int e = 0; e < EV; ++e) acc[e] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    m = -INFINITY;
    l = 0.f;
    cut0 = term >= 1 ? 0xffff0000u : 0u;
    cut1 = term >= 2 ? 0xffff0000u : 0u;
  }

  // K rows of a tile -> LDS (rows past the end re-read the last one)
  __device__ __forceinline__ void load_k(const bf16_t* __restrict__ K, const TileRef& t,
                                         unsigned char* lds) {
    const bf16_t* base = K + t.row0 * D;
    const int r = lane / CPR, jj = lane % CPR;
#pragma unroll
    for (int i = 0; i < kTile / RPI; ++i) {
      const int row = i * RPI + r;
      const bf16_t* src = base + min(row, t.len - 1) * D + (jj ^ swz(row)) * 8;
      __builtin_amdgcn_global_load_lds(
          (const __attribute__((address_space(1))) void*)src,
          (__attribute__((address_space(3))) void*)(lds + i * 1024), 16, 0, 2 /* nt */);
    }
  }

  __device__ __forceinline__ void load_v(const bf16_t* __restrict__ V, const TileRef& t,
                                         VRow (&vr)[NV]) {
    const bf16_t* base = V + t.row0 * D + (lane & 15) * EV;
    const int r = lane >> 4;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const bf16_t* src = base + min(4 * i + r, t.len - 1) * D;
      if constexpr (EV == 8) {
        vr[i] = ld_stream(src);
      } else {
        typedef unsigned u32x2_t __attribute__((ext_vector_type(2)));
        const u32x2_t v = __builtin_nontemporal_load(reinterpret_cast<const u32x2_t*>(src));
        vr[i] = make_uint2(v.x, v.y);
      }
    }
  }

  // logits of the tile in LDS: s[st][j] is token 16 st + 4 j + grp, head col % G
  __device__ __forceinline__ void logits(const unsigned char* lds, f32x4_t (&s)[NS]) {
    const int row0 = 4 * (lane & 3) + ((lane & 15) >> 2), grp = lane >> 4;
#pragma unroll
    for (int st = 0; st < NS; ++st) s[st] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kb = 0; kb < KB; ++kb)
#pragma unroll
      for (int st = 0; st < NS; ++st) {
        const int row = 16 * st + row0;
        const bf16x8_t a = *reinterpret_cast<const bf16x8_t*>(
            lds + row * (D * 2) + (((kb * 4 + grp) ^ swz(row)) * 16));
        s[st] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, qb[kb], s[st], 0, 0, 0);
      }
  }

  // mask, online softmax; s becomes p
  __device__ __forceinline__ void softmax(const TileRef& t, f32x4_t (&s)[NS]) {
    const int grp = lane >> 4;
    if (t.len < kTile) {                   // uniform
#pragma unroll
      for (int st = 0; st < NS; ++st)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          s[st][j] = 16 * st + 4 * j + grp < t.len ? s[st][j] : -INFINITY;
    }
    if (G > 1 && (t.hmask & ((1u << G) - 1u)) != ((1u << G) - 1u)) {   // uniform
      const bool on = (t.hmask >> ((lane & 15) % G)) & 1u;
#pragma unroll
      for (int st = 0; st < NS; ++st)
#pragma unroll
        for (int j = 0; j < 4; ++j) s[st][j] = on ? s[st][j] : -INFINITY;
    }
    float mt = -INFINITY;
#pragma unroll
    for (int st = 0; st < NS; ++st)
#pragma unroll
      for (int j = 0; j < 4; ++j) mt = fmaxf(mt, s[st][j]);
    float lo, hi;
    xor_pair<16>(mt, lo, hi);
    mt = fmaxf(lo, hi);
    xor_pair<32>(mt, lo, hi);
    mt = fmaxf(lo, hi) * qs;
    const float mn = fmaxf(m, mt);
    const float mref = mn == -INFINITY ? 0.f : mn;
    if (__ballot(mn != m)) {               // some head's maximum grew
      const float scale = fast_exp2(m - mref);   // 0 on the head's first tile
      l *= scale;
#pragma unroll
      for (int e = 0; e < EV; ++e)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[e][j] *= scale;
      m = mn;
    }
    float sum = 0.f;                       // of this lane's 16 tokens
#pragma unroll
    for (int st = 0; st < NS; ++st)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        s[st][j] = fast_exp2(fmaf(s[st][j], qs, -mref));
        sum += s[st][j];
      }
    l += sum;
  }

  // acc += V^T P^T
  __device__ __forceinline__ void pv(const VRow (&vr)[NV], const f32x4_t (&p)[NS]) {
    constexpr float kTiny = 1.17549435e-38f;     // smallest normal number
#pragma unroll
    for (int h = 0; h < 2; ++h) {          // 32 tokens each
      uint32_t w[4], w2[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        uint32_t x[2], y[2];
#pragma unroll
        for (int z = 0; z < 2; ++z) {
          const float pz = p[2 * h + i / 2][2 * (i & 1) + z];
          float t = pz - __uint_as_float(__float_as_uint(pz) & cut0);
          if constexpr (kTerms == 3) t -= __uint_as_float(__float_as_uint(t) & cut1);
          x[z] = __float_as_uint(__builtin_amdgcn_fmed3f(t, pz, kTiny));
          if constexpr (kTerms == 2) {     // term 2, in the first G columns
            float u = pz - __uint_as_float(__float_as_uint(pz) & 0xffff0000u);
            u -= __uint_as_float(__float_as_uint(u) & 0xffff0000u);
            y[z] = __float_as_uint(__builtin_amdgcn_fmed3f(cut0 ? 0.f : u, pz, kTiny));
          }
        }
        // upper halves of two words: a truncated bf16 pair
        w[i] = __builtin_amdgcn_perm(x[1], x[0], 0x07060302u);
        if constexpr (kTerms == 2) w2[i] = __builtin_amdgcn_perm(y[1], y[0], 0x07060302u);
      }
      const uint4 b = make_uint4(w[0], w[1], w[2], w[3]);
#pragma unroll
      for (int e = 0; e < EV; ++e) {
        uint32_t a[4];
#pragma unroll
        for (int i = 0; i < 4; ++i)
          a[i] = __builtin_amdgcn_perm(word(vr[8 * h + 2 * i + 1], e / 2),
                                       word(vr[8 * h + 2 * i], e / 2),
                                       (e & 1) ? 0x07060302u : 0x05040100u);
        const bf16x8_t av = __builtin_bit_cast(bf16x8_t, make_uint4(a[0], a[1], a[2], a[3]));
        acc[e] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, __builtin_bit_cast(bf16x8_t, b),
                                                         acc[e], 0, 0, 0);
        if constexpr (kTerms == 2)
          acc[e] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
              av, __builtin_bit_cast(bf16x8_t, make_uint4(w2[0], w2[1], w2[2], w2[3])), acc[e], 0,
              0, 0);
      }
    }
  }
  __device__ static __forceinline__ uint32_t word(const uint4& v, int i) {
    return i == 0 ? v.x : i == 1 ? v.y : i == 2 ? v.z : v.w;
  }
  __device__ static __forceinline__ uint32_t word(const uint2& v, int i) {
    return i == 0 ? v.x : v.y;
  }

  // tiles first, first + step, ... < end of at(i); wave-uniform call; lds:
  // the wave's own kLdsBytes
  template <typename At>
  __device__ __forceinline__ void run(const bf16_t* K, const bf16_t* V, int first, int end,
                                      int step, unsigned char* lds, At&& at) {
    if (first >= end) return;
    VRow vr[NV];
    TileRef t = at(first);
    load_k(K, t, lds);
    load_v(V, t, vr);
    for (int i = first;; i += step) {
      const bool more = i + step < end;
      TileRef nt{};
      if (more) nt = at(i + step);
      f32x4_t s[NS];
      logits(lds, s);
      // the logits' reads of LDS are over before the next rows may land there
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0)
      __builtin_amdgcn_sched_barrier(0);
      if (more) load_k(K, nt, lds);
      softmax(t, s);
      pv(vr, s);
      if (!more) break;
      load_v(V, nt, vr);
      t = nt;
    }
  }

  // the wave's totals (see TileVec::finish)
  __device__ __forceinline__ void finish(float* wacc, float* wm, float* wl) {
    const int col = lane & 15, grp = lane >> 4;
    l = xor_sum<16>(l);
    l = xor_sum<32>(l);
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int e0 = 0; e0 < EV; e0 += 4) {
        float a[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          // the lane of term 1 is G lanes up in the row, of term 2 another G
          const float v = acc[e0 + e][j];
          a[e] = v + dpp_f<kDppRowRor0 + 16 - G>(v);
          if constexpr (kTerms == 3) a[e] += dpp_f<kDppRowRor0 + 16 - 2 * G>(v);
        }
        if (col < G)
          *reinterpret_cast<float4*>(&wacc[col * D + EV * (4 * grp + j) + e0]) =
              make_float4(a[0], a[1], a[2], a[3]);
      }
    if (grp == 0 && col < G) { wm[col] = m; wl[col] = l; }
  }
};

template <typename T, int D, int G>
using Tile = typename std::conditional<sizeof(T) == 2, TileMfma<D, G>, TileVec<D, G>>::type;
template <typename T, int D, int G>
using AttendTile = typename std::conditional<sizeof(T) == 2, TileMfma<D, G>,
                                             TileVec<D, G, D == 128 && G <= 2 ? 32 : 16>>::type;

// ---------------------------------------------------------------------------
// phi(q) of a group's heads (Eq. 4)
// ---------------------------------------------------------------------------
// 16 lanes per Omega row, 4 rows per wave and pass: a lane multiplies its
// D / 16 dims (bf16 caches: v_dot2_f32_bf16 on the raw pairs, an fp32 Omega
// rounded to bf16 first; fp32 caches: an fma chain), and the NP * G sums of a
// lane's passes and heads are transpose-reduced over the 16 lanes, so each
// lane ends with one sum per 16 and the exponent, exp2 and store run once per
// feature and head. (A 16-lane reduction and an exp2 in every lane per feature
// and head, the form before, is three times the instructions. The matrix
// cores take fewer still, but their sums put the scores of a 512K context off
// by 1e-6 where these are off by 2e-7, and reading Omega in operand layout, 16
// rows per load, was 1 us slower.)
template <typename T, int D, int G, int NP>
struct PhiRows {
  static constexpr bool HALF = sizeof(T) == 2;
  static constexpr int QPL = D / 16;       // dims per lane
  static constexpr int W = HALF ? QPL / 2 : QPL;   // words of q or Omega per lane
  static constexpr int NVAL = NP * G;      // sums per lane
  // NP passes of Omega rows in flight: raw words, as stored (BF: bf16)
  template <bool BF> struct Om { uint32_t w[NP][BF ? W : QPL]; };
  uint32_t qw[G][W];
  float nrm;                               // |q|^2 s2 of the head this lane ends with

  template <int NWORD>
  __device__ static __forceinline__ void load_words(uint32_t (&w)[NWORD], const void* src) {
    if constexpr (NWORD == 2) {
      const uint2 u = *static_cast<const uint2*>(src);
      w[0] = u.x; w[1] = u.y;
    } else {
#pragma unroll
      for (int i = 0; i < NWORD / 4; ++i) {
        const uint4 u = static_cast<const uint4*>(src)[i];
        w[4 * i] = u.x; w[4 * i + 1] = u.y; w[4 * i + 2] = u.z; w[4 * i + 3] = u.w;
      }
    }
  }
  // pass p reads row `row` + p * step (row: this lane's row of pass 0)
  template <bool BF>
  __device__ static __forceinline__ void load(Om<BF>& om, const void* omega, int row, int step,
                                              int lane) {
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      const int at = (row + p * step) * D + (lane & 15) * QPL;
      if constexpr (BF) load_words(om.w[p], static_cast<const bf16_t*>(omega) + at);
      else load_words(om.w[p], static_cast<const float*>(omega) + at);
    }
  }
  __device__ __forceinline__ void load_q(const T* q0, int lane) {
#pragma unroll
    for (int g = 0; g < G; ++g) load_words(qw[g], q0 + g * D + (lane & 15) * QPL);
  }
  // the four bits of jj in reverse order
  __device__ static __forceinline__ int reversed(int jj) {
    return ((jj & 1) << 3) | ((jj & 2) << 1) | ((jj & 4) >> 1) | (jj >> 3);
  }
  __device__ static __forceinline__ float dot(uint32_t a, uint32_t b, float c) {
    if constexpr (HALF)
      return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2v_t, a),
                                             __builtin_bit_cast(bf16x2v_t, b), c, false);
    else
      return fmaf(__uint_as_float(a), __uint_as_float(b), c);
  }
  __device__ __forceinline__ void norm(float s2, int lane) {
    constexpr int GRP = NVAL < 16 ? NVAL : 16;
    const int mine = reversed(lane & 15) / (16 / GRP);   // its sum (features)
#pragma unroll
    for (int g = 0; g < G; ++g) {
      float sq = 0.f;
#pragma unroll
      for (int i = 0; i < W; ++i) sq = dot(qw[g][i], qw[g][i], sq);
      sq = row_sum(sq) * s2;
      nrm = g == 0 || mine % G == g ? sq : nrm;
    }
  }
  // phi of the loaded rows: put(head, pass, value)
  template <bool BF, typename Put>
  __device__ __forceinline__ void features(const Om<BF>& om, float s1, float inv_sqrt_n, int lane,
                                           Put&& put) {
    constexpr int GRP = NVAL < 16 ? NVAL : 16;     // sums per transpose
    const int jj = lane & 15;
    float v[NVAL];
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      uint32_t w[W];
#pragma unroll
      for (int i = 0; i < W; ++i) {
        if constexpr (BF || !HALF) w[i] = om.w[p][i];
        else w[i] = f32_to_bf16(__uint_as_float(om.w[p][2 * i])) |
                    (f32_to_bf16(__uint_as_float(om.w[p][2 * i + 1])) << 16);
      }
#pragma unroll
      for (int g = 0; g < G; ++g) {
        float a = 0.f;
#pragma unroll
        for (int i = 0; i < W; ++i) a = dot(w[i], qw[g][i], a);
        v[p * G + g] = a;
      }
    }
#pragma unroll
    for (int q = 0; q < NVAL / GRP; ++q) {
      // lowest lane bit first, so that every sum adds its 16 terms in the
      // order of row_sum; lanes that share a sum keep adding
      float x[GRP];
#pragma unroll
      for (int i = 0; i < GRP; ++i) x[i] = v[q * GRP + i];
      auto step = [&](auto mask, auto count) {
        constexpr int M = decltype(mask)::value, C = decltype(count)::value;
        if constexpr (C > 1) {
          const bool up = (lane & M) != 0;
#pragma unroll
          for (int i = 0; i < C / 2; ++i) {
            const float lo = x[i], hi = x[i + C / 2];
            x[i] = (up ? hi : lo) + row_xor<M>(up ? lo : hi);
          }
        } else {
          x[0] += row_xor<M>(x[0]);
        }
      };
      step(std::integral_constant<int, 1>{}, std::integral_constant<int, GRP>{});
      step(std::integral_constant<int, 2>{}, std::integral_constant<int, GRP / 2>{});
      step(std::integral_constant<int, 4>{}, std::integral_constant<int, GRP / 4>{});
      step(std::integral_constant<int, 8>{}, std::integral_constant<int, GRP / 8>{});
      // the first lane bit chose the upper half of the sums, and so on
      const int rev = reversed(jj);
      const int at = q * GRP + rev / (16 / GRP);
      const float ph = fast_exp2(fmaf(x[0], s1, -nrm)) * inv_sqrt_n;
      if (rev % (16 / GRP) == 0) put(at % G, at / G, ph);
    }
  }
};

// decode path shared by the fused kernel and its select-only instantiation
// k_decode_fused modes: the whole step; the selection only (select path);
// the step from scores the split path's kernels computed (scored path)
constexpr int kFusedFull = 0;
constexpr int kFusedSelect = 1;
constexpr int kFusedScored = 2;
constexpr int kFusedWaves = 8;
constexpr int kFusedMaxG = 4;
constexpr int kScoredMaxG = 8;     // bf16 caches (4 for fp32 ones)

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
// text of the last HIP error seen by this thread
extern thread_local char g_last_error[256];
// phase-clock buffer of the fused kernel's launches from this thread (null:
// off) and the number of workgroups it has room for
extern thread_local uint64_t* g_clock;
extern thread_local int g_clock_max;

// ---- launch helper with optional per-kernel event timing -----------------
// While profiling is enabled on a host thread, every launch goes through
// hipExtLaunchKernelGGL with a start/stop event pair, so the recorded times
// bracket exactly that kernel's execution on its stream.
// Read records return their events to a pool, so a profiled pass that
// follows another creates no events (event creation is host work that would
// otherwise slow the launches being timed).
struct Profiler {
  bool on = false;
  struct Rec { int kind; hipEvent_t a, b; };
  std::vector<Rec> recs;
  std::vector<hipEvent_t> pool;
  bool take(hipEvent_t* e) {
    if (!pool.empty()) { *e = pool.back(); pool.pop_back(); return true; }
    return hipEventCreate(e) == hipSuccess;
  }
};
extern thread_local Profiler g_prof;

template <typename F, typename... Args>
inline void launch(int kind, F kern, dim3 grid, dim3 block, size_t shm, hipStream_t st,
            Args... args) {
  if (g_prof.on) {
    hipEvent_t a = nullptr, b = nullptr;
    if (g_prof.take(&a)) {
      if (g_prof.take(&b)) {
        hipExtLaunchKernelGGL(kern, grid, block, (uint32_t)shm, st, a, b, 0u, args...);
        g_prof.recs.push_back({kind, a, b});
        return;
      }
      g_prof.pool.push_back(a);
    }
  }
  hipLaunchKernelGGL(kern, grid, block, shm, st, args...);
}

struct Shape {
  int B, Hq, Hkv, G, d, n, c, w, n_sink, per_head;
  int64_t cap, s_cap;
  radar_dtype dt;
  bool obf;                                // Omega stored as bf16
};

inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }
inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

struct WsLayout {
  size_t scores, uni, ucnt, part, total;
  int umax, maxwg, tiles_per_seg;
};

// RADAR_EHIP with the HIP error text recorded, or RADAR_OK
radar_status launch_status();

// compute units of the current device
int num_cu();

// K / V rows after the n_sink sink rows of the first (b, kv head): the
// kernels address segments and the window from there
// K / V rows after the n_sink sink rows of the first (b, kv head): the
// kernels address segments and the window from there
template <typename P>
P* after_sinks(const Shape& s, P* p) {
  const size_t esz = s.dt == RADAR_BF16 ? 2 : 4;
  using B = typename std::conditional<std::is_const<P>::value, const unsigned char,
                                      unsigned char>::type;
  return reinterpret_cast<P*>(reinterpret_cast<B*>(p) + (size_t)s.n_sink * s.d * esz);
}

// Split of the attention work (see attend_grid).
struct AttendGrid {
  int grid_x, tpw;
};

// ---- launchers provided by the units ---------------------------------------
// build.hip: segment summaries of segments [seg_first, seg_first + seg_count)
// of every (b, kv head), or with pos the per-sequence segment closes; K
// starts after the sinks
radar_status launch_build(const Shape& s, const void* K, const void* omega,
                          float* summ, int seg_first, int seg_count,
                          const int64_t* pos, hipStream_t st);

// split.hip: the split path's stages
// phi(q) and Eq. 6 scores of up to n_cand candidates of every query head into
// scores_of(base), in ScorePlan's slices; base: the workspace's score array
struct ScorePlan {
  int nsl;             // slices of the features; 0: two kernels, one slice
  int64_t stride;      // floats between them
};
ScorePlan score_plan(const Shape& s, int n_cand);
// (the two kernels' phi(q) lies before the scores)
inline float* scores_of(const Shape& s, float* base, const ScorePlan& sp) {
  return base + (sp.nsl == 0 ? (int64_t)s.B * s.Hq * s.n : 0);
}
void launch_scores(const Shape& s, const void* q, const void* omega, const float* summ,
                   float* base, int n_cand, const ScorePlan& sp, const SeqArgs& sa,
                   hipStream_t st);
// ln(beta) of candidates [0, n_cand) into rows of nc_cap scores; with_rest
// also the mass of the window and sinks at index n_cand
void launch_segment_mass(const Shape& s, const void* q, const void* K, float* scores,
                         int n_cand, const SeqArgs& sa, int nc_cap, bool with_rest,
                         hipStream_t st);
void launch_topk_union(const Shape& s, const float* scores, const ScorePlan& sp,
                       const SeqArgs& sa, int* uni, int* ucnt, int umax, int32_t* selected,
                       float* sel_scores, const AppendArgs& ap, hipStream_t st);
void launch_union_given(const Shape& s, const int32_t* given, int given_k,
                        const SeqArgs& sa, int* uni, int* ucnt, int umax,
                        hipStream_t st);
int64_t extra_tiles(const Shape& s, const SeqArgs& sa);
AttendGrid attend_grid(const Shape& s, const WsLayout& L, int u_bound, int64_t extra);
radar_status launch_attend(const Shape& s, const void* q, const void* K,
                           const void* V, const AttendGrid& ag, const SeqArgs& sa,
                           void* out, unsigned char* w, const WsLayout& L,
                           hipStream_t st);
void launch_combine_any(const Shape& s, const float* part, const int* ucnt, void* out,
                        const SeqArgs& sa, const WsLayout& L, int tpw, int fixed_nwg,
                        int partials_per_head, hipStream_t st);

// fused.hip (one unit per feature count n): the fused decode kernel, or with
// sel its select-only instantiation that hands the union to the split path
struct FusedArgs {
  const Shape* s;
  const void *q, *K, *V, *omega;
  const float* summ;
  SeqArgs sa;
  void* out;
  int32_t* selected;
  float* sel_scores;
  int *uni_out, *ucnt_out;
  int umax;
  AppendArgs ap;
  int R;
  float* part;
  int maxwg;
  hipStream_t st;
  const float* gscores;    // scored path: [B][Hq][nc_cap] Eq. 6 scores
  int nc_cap;
  ScorePlan sp;
};
radar_status launch_fused_n64(const FusedArgs& a, bool sel);
radar_status launch_fused_n128(const FusedArgs& a, bool sel);
radar_status launch_fused_n256(const FusedArgs& a, bool sel);
radar_status launch_fused_n512(const FusedArgs& a, bool sel);
radar_status launch_fused_n1024(const FusedArgs& a, bool sel);
radar_status launch_fused_n2048(const FusedArgs& a, bool sel);
// (fused_n64 unit) the fused kernel from phase 3 on, over gscores
radar_status launch_fused_scored(const FusedArgs& a);

}  // namespace radar_impl

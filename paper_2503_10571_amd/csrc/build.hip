// Index build (Eq. 4 and Eq. 5): k_build_bf16 (bf16 keys) and k_build_f32
// (fp32 keys) and their launchers. The segment close of an append runs the
// same kernel on one segment, so appends and rebuilds agree bit for bit.
#include "radar_impl.h"

namespace radar_impl {

// ---------------------------------------------------------------------------
// k_build_f32: segment summaries (Eq. 4, Eq. 5) of fp32 keys
// ---------------------------------------------------------------------------
// Work item = one (b, kv head, segment) and one slice of 64*FT features.
// Wave w of the workgroup owns features [w*16*FT, (w+1)*16*FT) of the slice
// and keeps that slice of Omega resident in registers as MFMA B operands for
// the whole kernel. Keys stream through two LDS buffers in tiles of 64 tokens
// (register-prefetched one tile ahead, one barrier per tile); every wave
// multiplies each 16-token sub-tile with its Omega slice on the matrix cores,
// applies exp2(acc * s1 - |k|^2 * s2) and adds the result into per-lane
// column sums. At the segment's end the sums are reduced across the four
// row groups of the MFMA output and scaled by 1 / (c sqrt(n)).
//
// MFMA operand layout (v_mfma_f32_16x16x4_f32; the bf16 16x16x32 one below
// holds eight k-slots per lane instead of one):
//   A (keys):    lane l supplies row (l & 15), k-slots of group (l >> 4)
//   B (Omega^T): lane l supplies column (l & 15), same k-slots
//   D:           lane l holds rows 4*(l >> 4) + j, j < 4, column (l & 15)
// The k-slot -> head-dim map is the same for A and B, so the dot products
// are the same whatever order the hardware sums them in. The fp32 matrix
// rate (1/16 of bf16) bounds this kernel, not its staging.
template <int D, int FT>
__global__ __launch_bounds__(256) void k_build_f32(
    const float* __restrict__ K, const float* __restrict__ omega, float* __restrict__ summ,
    int n, int c, int64_t cap, int64_t s_cap, int seg_first, int seg_count, int64_t n_items, float s1, float s2,
    float out_scale, int64_t kv_head_stride_rows,
    const int64_t* __restrict__ pos, int Hkv, int n_sink) {
  constexpr int TL = kTile;                // keys per LDS tile
  constexpr int KB = D / 4;                // MFMA steps per product
  constexpr int kPitch = D * 4 + 16;       // LDS row pitch in bytes
  constexpr int CPR = D / 4;               // 16-byte chunks per row
  constexpr int CPT = TL * CPR / 256;      // chunks per thread
  static_assert(CPT >= 1 && (256 % CPR) == 0, "tile shape");

  __shared__ __attribute__((aligned(16))) unsigned char tile_lds[2][TL * kPitch];
  __shared__ float nrm_lds[2][TL];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int col = lane & 15;
  const int grp = lane >> 4;
  const int fbase = blockIdx.y * (64 * FT) + wave * (16 * FT);

  // Omega slice -> B fragments (resident for the whole kernel)
  float bfrag[FT][KB];
#pragma unroll
  for (int f = 0; f < FT; ++f) {
    const int64_t orow = (int64_t)(fbase + f * 16 + col) * D;
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) {
      bfrag[f][kb] = omega[orow + kb * 4 + grp];
    }
  }

  const int ntiles = (c + TL - 1) / TL;
  float psum[FT];
#pragma unroll
  for (int f = 0; f < FT; ++f) psum[f] = 0.f;

  // Segment of an item (one (b, kv head, segment); 32-bit arithmetic, item
  // counts stay below 2^31): seg_first + item % seg_count, or, with pos
  // (item = (b, kv head), one per-sequence segment close), the segment that
  // row pos[b] completes, -1 if it completes none. Rows count from the
  // first row after the n_sink sinks, where the K pointer starts.
  auto seg_of = [&](int64_t it) -> int {
    const uint32_t u = (uint32_t)it;
    if (!pos) return seg_first + (int)(u % (uint32_t)seg_count);
    const int64_t p = pos[u / (uint32_t)Hkv];
    const int64_t r = p - n_sink;
    if (p >= cap || r < 0 || (r + 1) % c != 0) return -1;
    return (int)((r + 1) / c - 1);
  };
  // first active item at or after it on this workgroup's stride
  auto next_active = [&](int64_t it) -> int64_t {
    while (it < n_items && seg_of(it) < 0) it += gridDim.x;
    return it;
  };
  // base row pointer of an item, computed once per segment
  auto item_base = [&](int64_t it) -> const float* {
    const uint32_t bh = (uint32_t)it / (uint32_t)seg_count;
    return K + ((int64_t)bh * kv_head_stride_rows + (int64_t)seg_of(it) * c) * D;
  };

  uint4 pre[CPT];
  int pre_valid = 0;
  // tile tl of the item whose rows start at `base`
  auto fetch = [&](const float* base, int tl_) {
    pre_valid = min(TL, c - tl_ * TL);
    const float* src = base + (int64_t)tl_ * TL * D;
#pragma unroll
    for (int p = 0; p < CPT; ++p) {
      const int ci = p * 256 + tid;
      // rows past the segment re-read its last row; they are masked out
      // of the sums below
      const int row = min(ci / CPR, pre_valid - 1), ch = ci % CPR;
      pre[p] = ld_stream(reinterpret_cast<const unsigned char*>(src + (int64_t)row * D) +
                         ch * 16);
    }
  };
  // registers -> LDS buffer `buf`, with |k|^2 * s2 per row: the CPR chunks
  // of a row sit in CPR consecutive lanes, summed by DPP row reductions
  auto stage = [&](int buf) {
    unsigned char* tb = tile_lds[buf];
#pragma unroll
    for (int p = 0; p < CPT; ++p) {
      const int ci = p * 256 + tid;
      const int row = ci / CPR, ch = ci % CPR;
      *reinterpret_cast<uint4*>(tb + row * kPitch + ch * 16) = pre[p];
      float sq = 0.f;
      float e[4];
      unpack16<float>(pre[p], e);
#pragma unroll
      for (int i = 0; i < 4; ++i) sq = fmaf(e[i], e[i], sq);
      sq = row_sum(sq);
      if constexpr (CPR == 32) sq = xor_sum<16>(sq);
      if (ch == 0) nrm_lds[buf][row] = sq * s2;
    }
  };

  // 16-token sub-tiles of the tile in `buf`; FULL: no rows to mask
  auto compute = [&](int buf, int valid, auto full_tag) {
    constexpr bool FULL = decltype(full_tag)::value;
    const unsigned char* tb = tile_lds[buf];
#pragma unroll
    for (int st = 0; st < TL / 16; ++st) {
      if (!FULL && st * 16 >= valid) break;
      float afrag[KB];
      const unsigned char* arow = tb + (st * 16 + col) * kPitch;
#pragma unroll
      for (int kb = 0; kb < KB; ++kb) {
        afrag[kb] = *reinterpret_cast<const float*>(arow + (kb * 4 + grp) * 4);
      }
      float nb[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) nb[j] = nrm_lds[buf][st * 16 + grp * 4 + j];
      // head-dim block outer, feature tile inner: FT independent
      // accumulation chains keep the matrix pipe busy
      f32x4_t acc[FT];
#pragma unroll
      for (int f = 0; f < FT; ++f) acc[f] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int kb = 0; kb < KB; ++kb)
#pragma unroll
        for (int f = 0; f < FT; ++f) {
          acc[f] = __builtin_amdgcn_mfma_f32_16x16x4f32(afrag[kb], bfrag[f][kb], acc[f], 0, 0, 0);
        }
#pragma unroll
      for (int f = 0; f < FT; ++f)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const float v = fast_exp2(fmaf(acc[f][j], s1, -nb[j]));
          if (FULL) psum[f] += v;
          else psum[f] += (st * 16 + grp * 4 + j < valid) ? v : 0.f;
        }
    }
  };

  // Pipeline, one barrier per tile: tile i is multiplied from one LDS buffer
  // while tile i+1 is in flight to registers; after the multiply the
  // registers go to the other buffer.
  int64_t item = next_active(blockIdx.x);
  int tl = 0, buf = 0;
  const float* base = nullptr;
  if (item < n_items) {
    base = item_base(item);
    fetch(base, 0);
    stage(0);
  }
  int valid = pre_valid;
  __syncthreads();
  while (item < n_items) {
    int64_t nitem = item;
    int ntl = tl + 1;
    const float* nbase = base;
    if (ntl == ntiles) {
      nitem = next_active(nitem + gridDim.x);
      ntl = 0;
      if (nitem < n_items) nbase = item_base(nitem);
    }
    const bool more = nitem < n_items;
    if (more) fetch(nbase, ntl);

    if (valid == TL) compute(buf, valid, std::true_type{});
    else compute(buf, valid, std::false_type{});

    if (tl == ntiles - 1) {                // segment complete
      const int64_t bh = (uint32_t)item / (uint32_t)seg_count;
      const int64_t sg = seg_of(item);
      float* dst = summ + (bh * s_cap + sg) * n + fbase;
#pragma unroll
      for (int f = 0; f < FT; ++f) {
        float v = psum[f];
        v = xor_sum<16>(v);
        v = xor_sum<32>(v);
        if (lane < 16) dst[f * 16 + col] = v * out_scale;
        psum[f] = 0.f;
      }
    }
    if (more) stage(buf ^ 1);
    __syncthreads();
    buf ^= 1;
    valid = pre_valid;
    item = nitem;
    tl = ntl;
    base = nbase;
  }
}

// ---------------------------------------------------------------------------
// k_build_bf16: the summaries of bf16 keys, one wave per segment
// ---------------------------------------------------------------------------
// Work item = one (b, kv head, segment) for one slice of 16 * NF features,
// done by one wave from its first key to its last: the slice of Omega sits
// in LDS as MFMA B fragments (written once per workgroup), the wave's keys
// come straight from memory into registers as A fragments, 64 at a time, and
// the waves never meet after the Omega barrier. Feature tile f + 1 is
// multiplied while the exp2 epilogue of tile f runs (two accumulator sets);
// B fragments are read one tile ahead.
// With SPLIT (few long segments, where one wave's chain of blocks would be the
// whole call) a workgroup takes an item: its waves take the 64-key blocks in
// turn, and a segment's total adds the block sums in block order, as a wave
// that walks the segment alone does, so both forms give the same bits.
//
// What bounds it is the matrix and vector work of a SIMD together. A 16x16 tile
// of keys and features at d = 128 is 64 cycles on the matrix pipe and 96 of
// vector issue (four elements per lane: exp2 at quarter rate 64, fma and add 16
// each); a SIMD takes 135 per tile at 256 features (33.5 M keys in 2.38 ms at the
// 1.86 GHz that it runs at; the matrix pipe is busy 47% of them), however the
// two are interleaved, by hand or by the compiler, to within 3%. Keys staged
// through LDS and shared by four waves, with a barrier per 128 keys (the layout
// before this one), took 2.71 ms; 615 -> 535 us for 4.2 M keys at n = 512 and 94
// -> 67 us for 131 K keys at n = 2048. Fetching the next block ahead (n <= 256,
// where the registers allow it) is worth 2%.
// HOST: the keys lie in host memory (see fetch).
template <int D, int NF, int NW, bool SPLIT, bool HOST>
__global__ __launch_bounds__(64 * NW, 2) void k_build_bf16(
    const bf16_t* __restrict__ K, const void* __restrict__ omega, bool obf,
    float* __restrict__ summ, int n, int c, int64_t cap, int64_t s_cap,
    int seg_first, int seg_count, uint32_t item0, uint32_t n_items, float s1, float s2,
    float out_scale, const int64_t* __restrict__ pos, int Hkv, int n_sink) {
  constexpr int KB = D / 32;               // MFMA steps per product
  constexpr int NS = 4;                    // 16-key sub-tiles per block
  constexpr bool kAhead = NF <= 16;        // registers for two blocks of keys
  __shared__ __attribute__((aligned(16))) uint4 om_lds[NF * KB * 64];
  __shared__ __attribute__((aligned(16))) float nrm_lds[NW][NS * 16];
  // SPLIT: a round's block sums, two rounds' worth
  __shared__ float bsum[SPLIT ? 2 : 1][SPLIT ? NW : 1][SPLIT ? NF : 1][64];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int col = lane & 15;
  const int grp = lane >> 4;
  const int fbase = blockIdx.y * (16 * NF);
  const uint32_t stride = SPLIT ? gridDim.x : gridDim.x * NW;

  // the segment of an item: seg_first + item % seg_count, or, with pos (item
  // = (b, kv head), one per-sequence segment close), the segment that row
  // pos[b] completes, -1 if it completes none
  auto seg_of = [&](uint32_t it) -> int {
    if (!pos) return seg_first + (int)(it % (uint32_t)seg_count);
    const int64_t p = pos[it / (uint32_t)Hkv];
    const int64_t r = p - n_sink;
    if (p >= cap || r < 0 || (r + 1) % c != 0) return -1;
    return (int)((r + 1) / c - 1);
  };
  auto next_active = [&](uint32_t it) -> uint32_t {
    while (it < n_items && seg_of(it) < 0) it += stride;
    return it;
  };
  auto item_base = [&](uint32_t it) -> const bf16_t* {
    return K + ((int64_t)(it / (uint32_t)seg_count) * cap + (int64_t)seg_of(it) * c) * D;
  };

  // items [item0, n_items) of the call
  uint32_t item = next_active(item0 + (SPLIT ? blockIdx.x : blockIdx.x * NW + wave));
  // a workgroup without a segment to close leaves before it reads Omega
  if (pos && !__syncthreads_or(item < n_items)) return;

  // key blocks: lane (row col, k-slot group grp) of sub-tile st holds bytes
  // kb * 64 + grp * 16 .. + 16 of key st * 16 + col; keys past the segment
  // re-read its last one and are masked by their norm
  uint32_t touched = 0;
  auto fetch = [&](uint4 (&A)[NS][KB], const bf16_t* base, int off) {
    // HOST: the loads below ask for half a line each, and the host link gives
    // 45 to 53 GB/s; a word of both halves of every line first asks for whole
    // ones (56 GB/s: 1.07 GB of keys 22.1 -> 19.1 ms, 268 MB 5.65 -> 4.79)
    if constexpr (HOST) {
#pragma unroll
      for (int i = 0; i < D / 32; ++i) {
        const int half = i * 64 + lane;    // of the block's lines
        const int row = min(off + half / (D / 32), c - 1);
        touched ^= *reinterpret_cast<const uint32_t*>(base + (int64_t)row * D + half % (D / 32) * 32);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int st = 0; st < NS; ++st) {
      const int row = min(off + st * 16 + col, c - 1);
      const bf16_t* src = base + (int64_t)row * D + grp * 8;
#pragma unroll
      for (int kb = 0; kb < KB; ++kb)
        A[st][kb] = *reinterpret_cast<const uint4*>(src + kb * 32);
    }
  };

  uint4 keys[NS][KB];
  const bf16_t* base = nullptr;
  if (item < n_items) {
    base = item_base(item);
    const int first = SPLIT ? wave * NS * 16 : 0;
    if (first < c) fetch(keys, base, first);
  }

  // Omega slice -> B fragments in LDS: fragment (f, kb), lane (col, grp):
  // dims kb * 32 + grp * 8 .. + 8 of feature f * 16 + col
  for (int i = tid; i < NF * KB * 64; i += NW * 64) {
    const int f = i / (KB * 64), kb = (i / 64) % KB, ln = i & 63;
    const int64_t i0 = (int64_t)(fbase + f * 16 + (ln & 15)) * D + kb * 32 + (ln >> 4) * 8;
    uint4 u;
    if (obf) {
      u = *reinterpret_cast<const uint4*>(static_cast<const bf16_t*>(omega) + i0);
    } else {
      const float* src = static_cast<const float*>(omega) + i0;
      uint32_t w[4];
#pragma unroll
      for (int e = 0; e < 4; ++e)
        w[e] = f32_to_bf16(src[2 * e]) | (f32_to_bf16(src[2 * e + 1]) << 16);
      u = make_uint4(w[0], w[1], w[2], w[3]);
    }
    om_lds[i] = u;
  }
  __syncthreads();

  // ST sub-tiles of 16 keys, the first `valid` of them real; put(f, sum of
  // this lane's elements of feature tile f)
  auto block = [&](const uint4 (&A)[NS][KB], int valid, auto st_tag, auto&& put) {
    constexpr int ST = decltype(st_tag)::value;
    // |k|^2 s2 of the block's 64 keys: every lane sums its 16-byte chunks of
    // a key, the four k-slot groups are added, and LDS turns the column
    // order of the A operand into the row order of the products; a key past
    // the segment gets +inf, so its exp2 is 0
    float nrm = 0.f;
#pragma unroll
    for (int st = 0; st < ST; ++st) {
      float sq = 0.f;
#pragma unroll
      for (int kb = 0; kb < KB; ++kb) {
        const uint32_t w[4] = {A[st][kb].x, A[st][kb].y, A[st][kb].z, A[st][kb].w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const bf16x2v_t v = __builtin_bit_cast(bf16x2v_t, w[i]);
          sq = __builtin_amdgcn_fdot2_f32_bf16(v, v, sq, false);
        }
      }
      sq = xor_sum<16>(sq);
      sq = xor_sum<32>(sq);
      nrm = grp == st ? sq : nrm;
    }
    nrm_lds[wave][lane] = lane < valid ? nrm * s2 : INFINITY;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    f32x4_t nb[ST];
#pragma unroll
    for (int st = 0; st < ST; ++st)
      nb[st] = *reinterpret_cast<const f32x4_t*>(&nrm_lds[wave][st * 16 + grp * 4]);

    uint4 b[2][KB];
    f32x4_t acc[2][ST];
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) b[0][kb] = om_lds[kb * 64 + lane];
    // slot q of tile f: product q of the tile's ST * KB, and of tile f - 1's
    // ST * 4 elements per lane the fma of element q, the exp2 of q - 1 and
    // the sum of q - 2 (so no instruction waits for the one before it)
    constexpr int NP = ST * KB, NE = ST * 4;
    constexpr int SLOTS = (NP > NE + 2 ? NP : NE + 2);
#pragma unroll
    for (int f = 0; f <= NF; ++f) {
      if (f + 1 < NF) {
#pragma unroll
        for (int kb = 0; kb < KB; ++kb)
          b[(f + 1) & 1][kb] = om_lds[((f + 1) * KB + kb) * 64 + lane];
      }
      float x[NE], sum = 0.f;
#pragma unroll
      for (int q = 0; q < SLOTS; ++q) {
        if (f < NF && q < NP) {
          const int kb = q / ST, st = q % ST;
          const f32x4_t zero = {0.f, 0.f, 0.f, 0.f};
          acc[f & 1][st] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
              __builtin_bit_cast(bf16x8_t, A[st][kb]),
              __builtin_bit_cast(bf16x8_t, b[f & 1][kb]), kb ? acc[f & 1][st] : zero, 0, 0, 0);
        }
        if (f > 0) {
          if (q < NE) x[q] = fmaf(acc[(f - 1) & 1][q / 4][q % 4], s1, -nb[q / 4][q % 4]);
          if (q >= 1 && q - 1 < NE) x[q - 1] = fast_exp2(x[q - 1]);
          if (q == 2) sum = x[0];
          if (q > 2 && q - 2 < NE) sum += x[q - 2];
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      if (f > 0) put(f - 1, sum);
    }
  };
  // a remainder of at most 32 keys takes half a block's products
  auto compute = [&](const uint4 (&A)[NS][KB], int valid, auto&& put) {
    if (valid > 32) block(A, valid, std::integral_constant<int, NS>{}, put);
    else block(A, valid, std::integral_constant<int, 2>{}, put);
  };

  if constexpr (SPLIT) {
    constexpr int OWN = (NF + NW - 1) / NW;      // feature tiles a wave adds up
    const int nblk = (c + NS * 16 - 1) / (NS * 16);
    int buf = 0;
    while (item < n_items) {               // workgroup-uniform
      const uint32_t nitem = next_active(item + stride);
      const bf16_t* nbase = nitem < n_items ? item_base(nitem) : nullptr;
      float tot[OWN];
#pragma unroll
      for (int i = 0; i < OWN; ++i) tot[i] = 0.f;
      for (int b0 = 0; b0 < nblk; b0 += NW, buf ^= 1) {
        const int blk = b0 + wave;
        uint4 next[NS][KB];
        const bool more = blk + NW < nblk;
        if (more) fetch(next, base, (blk + NW) * NS * 16);
        if (blk < nblk)
          compute(keys, c - blk * NS * 16, [&](int f, float v) { bsum[buf][wave][f][lane] = v; });
        if (more) {
#pragma unroll
          for (int st = 0; st < NS; ++st)
#pragma unroll
            for (int kb = 0; kb < KB; ++kb) keys[st][kb] = next[st][kb];
        }
        // (the buffer's readers of two rounds ago passed the last barrier)
        __syncthreads();
        const int here = min(NW, nblk - b0);
#pragma unroll
        for (int i = 0; i < OWN; ++i) {
          const int f = wave + i * NW;
          if (f < NF)
            for (int w = 0; w < here; ++w) tot[i] += bsum[buf][w][f][lane];
        }
      }
      if (nbase && wave < nblk) fetch(keys, nbase, wave * NS * 16);
      float* dst = summ + ((int64_t)(item / (uint32_t)seg_count) * s_cap + seg_of(item)) * n + fbase;
#pragma unroll
      for (int i = 0; i < OWN; ++i) {
        const int f = wave + i * NW;
        float v = tot[i];
        v = xor_sum<16>(v);
        v = xor_sum<32>(v);
        if (f < NF && lane < 16) dst[f * 16 + col] = v * out_scale;
      }
      item = nitem;
      base = nbase;
    }
    if (HOST && n < 0) summ[lane] = (float)touched;    // (never: keeps the loads)
    return;
  }

  float psum[NF];
#pragma unroll
  for (int f = 0; f < NF; ++f) psum[f] = 0.f;
  auto add = [&](int f, float v) { psum[f] += v; };

  // one block of `cur`; the next block's keys go to `nxt` (the same
  // registers where there is no room for two blocks)
  int off = 0;
  auto step = [&](uint4 (&cur)[NS][KB], uint4 (&nxt)[NS][KB]) {
    const uint32_t it = item;
    const int o = off;
    off += NS * 16;
    const bool last = off >= c;            // the segment's last block
    if (last) {
      item = next_active(item + stride);
      off = 0;
      if (item < n_items) base = item_base(item);
    }
    if (kAhead && item < n_items) fetch(nxt, base, off);
    compute(cur, c - o, add);
    if (!kAhead && item < n_items) fetch(nxt, base, off);
    if (last) {
      float* dst = summ + ((int64_t)(it / (uint32_t)seg_count) * s_cap + seg_of(it)) * n + fbase;
#pragma unroll
      for (int f = 0; f < NF; ++f) {
        float v = psum[f];
        v = xor_sum<16>(v);
        v = xor_sum<32>(v);
        if (lane < 16) dst[f * 16 + col] = v * out_scale;
        psum[f] = 0.f;
      }
    }
  };
  if constexpr (kAhead) {
    uint4 keys2[NS][KB];
    while (item < n_items) {
      step(keys, keys2);
      if (item >= n_items) break;
      step(keys2, keys);
    }
  } else {
    while (item < n_items) step(keys, keys);
  }
  if (HOST && n < 0) summ[lane] = (float)touched;      // (never: keeps the loads)
}

// Features per workgroup (16 nf), waves per workgroup and whether they share
// a segment, by the time the call should take: rounds of the persistent grid,
// times 64-key blocks per wave, times a wave's time per block with one wave per
// SIMD and with two (us, for nf = 2, 4, 8, 16, 32; a last round that fills at
// most half the chip runs at the first). At d = 128 below nf = 8 the keys' way
// through the L1 bounds a block, above it the products, so wide slices win where
// there is work for every wave (4.2 M keys at n = 512: 548 us at nf = 32, 705 at
// 8, 1852 at 2), narrow ones or split segments where there is not (36 segments
// of 647 keys at n = 1024: 19 us at nf = 16 split eight ways, 27 at nf = 4 and
// 138 at nf = 32 unsplit). At d = 64 a block costs less, and narrow slices lose
// less (624 segments of 426 keys at n = 2048: 112 us at nf = 8, 119 at 16 and 140
// at 16 split eight ways; d = 128, 825 of 470 at n = 1024: 108 at 32, 117 at 16
// and 130 at 16 split). The times are fitted to 781 shapes (8 to 20000 segments of
// 33 to 846 keys, both d, every n) in up to 13 forms each; the choice is within 2%
// of the fastest in the mean, one in twenty misses it by more than 5%. A feature's sum depends on
// none of this, so a segment close and a rebuild agree bit for bit.
struct BuildPlan {
  int nf, nw;
  bool split;
  uint32_t full;       // items of the grid's full rounds
  float us, full_us;   // estimates: all items, the full rounds alone
};
// f(plan) for every form of a build of `items` segments (32-bit arithmetic: a
// short append waits for this); link: only the form for keys in host memory (see
// launch_build_bf16_any)
template <typename F>
void each_build_plan(uint32_t items, int d, int n, int c, bool link, F&& f) {
  constexpr float kOne[2][5] = {{1.1f, 1.6f, 3.0f, 3.0f, 9.0f}, {1.9f, 2.2f, 3.2f, 5.8f, 14.0f}};
  constexpr float kTwo[2][5] = {{1.9f, 2.6f, 3.4f, 5.6f, 9.6f}, {2.4f, 3.7f, 4.5f, 6.9f, 12.1f}};
  const uint32_t cus = (uint32_t)num_cu(), nblk = ((uint32_t)c + 63) / 64;
  const float* one = kOne[d == 128], *two = kTwo[d == 128];
  // a remainder of at most 32 keys costs about half a block
  const float blocks = (float)nblk - (nblk * 64 - (uint32_t)c >= 32 ? 0.4f : 0.f);
  for (int i = 0; i < 5 && (32 << i) <= n; ++i) {
    const uint32_t nf = 2u << i, slices = (uint32_t)n / (16 * nf);
    if (link && i != 2 && (i > 2 || (64 << i) <= n)) continue;
    for (uint32_t split = 0; split < 3; ++split) {   // no, over 4 waves, over 8
      const uint32_t nw = split ? 4 * split : nf >= 16 ? 8 : 4;
      if (link ? split != 2 : split && (nf > 16 || nblk < 2 || (split == 2 && nblk <= 4))) continue;
      // (a split workgroup of nf = 16 has 96 KB of LDS or more)
      const bool alone = nw == 8 || (split && nf == 16);
      const uint32_t slots = std::max(1u, (alone ? 1 : 2) * cus / slices);
      const uint32_t groups = split ? items : (items + nw - 1) / nw;
      const uint32_t gx = std::min(groups, slots);
      const uint32_t full = groups / gx, rest = groups - full * gx;
      auto round = [&](uint32_t wgs) {     // of so many workgroups per slice
        const float t = nw == 4 && (alone || wgs * slices <= cus) ? one[i] : two[i];
        if (!split) return t * blocks;
        return (split == 1 ? 1.08f : 0.97f) * t * (float)((nblk + nw - 1) / nw) + 0.5f;
      };
      const float full_us = 0.1f * (float)nf + (float)full * round(gx);
      f(BuildPlan{(int)nf, (int)nw, split != 0, full * gx * (split ? 1 : nw),
                  full_us + (rest ? round(rest) : 0.f), full_us});
    }
  }
}
BuildPlan build_plan(uint32_t items, int d, int n, int c, bool link) {
  BuildPlan best{2, 4, false, 0, INFINITY, 0.f};
  each_build_plan(items, d, n, c, link, [&](const BuildPlan& p) { if (p.us < best.us) best = p; });
  return best;
}

// (60 ns a call)
bool on_host(const void* p) {
  hipPointerAttribute_t a{};
  if (hipPointerGetAttributes(&a, p) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  return a.type == hipMemoryTypeHost;
}

template <int D, int NF, int NW, bool SPLIT>
void launch_build_bf16(const Shape& s, const void* K, const void* omega, float* summ,
                       int seg_first, int seg_count, int64_t item0, int64_t items,
                       const int64_t* pos, bool host, hipStream_t st) {
  const int slices = s.n / (16 * NF);
  const int64_t resident = std::max<int64_t>(1, (8 / NW) * (int64_t)num_cu() / slices);
  const int64_t todo = items - item0;
  int64_t gx = std::min<int64_t>(SPLIT ? todo : ceil_div(todo, NW), resident);
  // workgroups go round the 8 XCDs in turn, so with a multiple of 8 a segment's
  // slices read it through one L2, and it comes over the host link once (27
  // segments of 724 keys in two slices: 101 us, 192 with 27 workgroups each)
  if (host) gx = ceil_div(gx, 8) * 8;
  const float s1 = kLog2e / std::pow((float)s.d, 0.25f);
  const float s2 = kLog2e / (2.f * std::sqrt((float)s.d));
  const float out_scale = 1.f / ((float)s.c * std::sqrt((float)s.n));
  launch(RADAR_K_BUILD,
         host ? k_build_bf16<D, NF, NW, SPLIT, true> : k_build_bf16<D, NF, NW, SPLIT, false>,
         dim3((unsigned)gx, (unsigned)slices), dim3(64 * NW), 0, st,
         reinterpret_cast<const bf16_t*>(K), omega, s.obf, summ, s.n, s.c, s.cap, s.s_cap,
         seg_first, seg_count, (uint32_t)item0, (uint32_t)items, s1, s2, out_scale, pos, s.Hkv,
         s.n_sink);
}

// items [item0, items) of the call by plan p
template <int D>
void launch_build_plan(const BuildPlan& p, const Shape& s, const void* K, const void* omega,
                       float* summ, int seg_first, int seg_count, int64_t item0, int64_t items,
                       const int64_t* pos, bool host, hipStream_t st) {
  auto go = [&](auto f, auto w, auto sp) {
    launch_build_bf16<D, decltype(f)::value, decltype(w)::value, decltype(sp)::value>(
        s, K, omega, summ, seg_first, seg_count, item0, items, pos, host, st);
  };
  auto go_f = [&](auto f) {
    constexpr int NF = decltype(f)::value;
    if constexpr (NF <= 16) {
      if (p.split && p.nw == 4) return go(f, std::integral_constant<int, 4>{}, std::true_type{});
      if (p.split) return go(f, std::integral_constant<int, 8>{}, std::true_type{});
    }
    // 8 waves share 64 or 128 KB of Omega where a wave takes a segment
    return go(f, std::integral_constant<int, NF >= 16 ? 8 : 4>{}, std::false_type{});
  };
  switch (p.nf) {
    case 2: return go_f(std::integral_constant<int, 2>{});
    case 4: return go_f(std::integral_constant<int, 4>{});
    case 8: return go_f(std::integral_constant<int, 8>{});
    case 16: return go_f(std::integral_constant<int, 16>{});
    default: return go_f(std::integral_constant<int, 32>{});
  }
}

template <int D>
radar_status launch_build_bf16_any(const Shape& s, const void* K, const void* omega,
                                   float* summ, int seg_first, int seg_count,
                                   const int64_t* pos, hipStream_t st) {
  const int64_t items = (int64_t)s.B * s.Hkv * seg_count;
  if (items == 0) return RADAR_OK;
  if (items >= ((int64_t)1 << 31)) return RADAR_EUNSUPPORTED;   // 32-bit item ids
  // Keys in host memory are asked for in whole lines (see fetch; from 2 MB, below
  // which it does not show) and come over the link once only where a segment's
  // slices read it through one L2 (see launch_build_bf16) at about the same time:
  // eight waves that share a segment keep its slices together, in slices of up to
  // 128 features (1.07 GB at n = 256 in segments of 256 keys: 19.1 ms, 56 GB/s;
  // 23.7 in one slice with a segment per wave, 38.3 with four waves; of 1500 keys:
  // 19.0, 25.5 in one split slice; 13 MB at n = 512 in segments of 64: 237 us, 275
  // in the form of device memory). Above n = 1024 these are too many slices where
  // segments are short, and the forms of device memory do as well or better
  // (n = 2048, 67 MB in segments of 33: 54 and 36 GB/s; 268 MB of 362: 56 and 51).
  const bool host = items * s.c * D * 2 > (2 << 20) && on_host(K);
  const bool link = host && s.n <= 1024;
  const BuildPlan p = build_plan((uint32_t)items, s.d, s.n, s.c, link);
  // A last round that is mostly empty goes to a launch of its own with the plan
  // for few items, where the estimates say that it pays for the launch, with the
  // plan whose full rounds and rest are the least then (2088 segments of 426
  // keys, d = 64, n = 256: 53 us, one launch 64; 524 of 426, d = 128, n = 1024:
  // 70 and 87). Not for closes: most of them have nothing to do.
  BuildPlan first = p, rest{};
  float us = 0.96f * p.us;
  if (!pos)
    each_build_plan((uint32_t)items, s.d, s.n, s.c, link, [&](const BuildPlan& f) {
      if (f.full == 0 || f.full >= items || f.full_us + 3.3f >= us) return;
      const BuildPlan r = build_plan((uint32_t)items - f.full, s.d, s.n, s.c, link);
      if (f.full_us + 3.3f + r.us < us) {
        us = f.full_us + 3.3f + r.us;
        first = f;
        rest = r;
      }
    });
  const int64_t full = rest.nf ? first.full : items;
  launch_build_plan<D>(first, s, K, omega, summ, seg_first, seg_count, 0, full, pos, host, st);
  if (full < items)
    launch_build_plan<D>(rest, s, K, omega, summ, seg_first, seg_count, full, items, pos, host, st);
  return launch_status();
}

template <int D, int FT>
radar_status launch_build_f32(const Shape& s, const void* K, const void* omega,
                              float* summ, int seg_first, int seg_count,
                              const int64_t* pos, hipStream_t st) {
  // features per workgroup = 64 * FT; FT capped so the resident Omega slice
  // stays at 128 VGPRs or fewer
  if constexpr (FT > 1) {
    if (64 * FT > s.n)
      return launch_build_f32<D, FT / 2>(s, K, omega, summ, seg_first, seg_count, pos, st);
  }
  const int slices = s.n / (64 * FT);
  const int64_t items = (int64_t)s.B * s.Hkv * seg_count;
  if (items == 0) return RADAR_OK;
  if (items >= ((int64_t)1 << 31)) return RADAR_EUNSUPPORTED;   // 32-bit item ids
  auto kern = k_build_f32<D, FT>;
  int per_cu = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, 256, 0) != hipSuccess || per_cu < 1)
    per_cu = 1;
  (void)hipGetLastError();
  const int64_t resident = (int64_t)per_cu * num_cu();
  const int64_t gx = std::min<int64_t>(items, std::max<int64_t>(1, resident / slices));
  const float s1 = kLog2e / std::pow((float)s.d, 0.25f);
  const float s2 = kLog2e / (2.f * std::sqrt((float)s.d));
  const float out_scale = 1.f / ((float)s.c * std::sqrt((float)s.n));
  launch(RADAR_K_BUILD, kern, dim3((unsigned)gx, (unsigned)slices), dim3(256), 0, st,
                     reinterpret_cast<const float*>(K), static_cast<const float*>(omega), summ, s.n, s.c, s.cap,
                     s.s_cap, seg_first, seg_count, items, s1, s2, out_scale, s.cap,
                     pos, s.Hkv, s.n_sink);
  return launch_status();
}

// K: the first row after the sinks (after_sinks); pos: per-sequence segment
// closes (seg_first / seg_count then 0 / 1)
radar_status launch_build(const Shape& s, const void* K, const void* omega,
                          float* summ, int seg_first, int seg_count,
                          const int64_t* pos, hipStream_t st) {
  if (s.dt == RADAR_BF16)
    return s.d == 64 ? launch_build_bf16_any<64>(s, K, omega, summ, seg_first, seg_count, pos, st)
                     : launch_build_bf16_any<128>(s, K, omega, summ, seg_first, seg_count, pos, st);
  return s.d == 64 ? launch_build_f32<64, 8>(s, K, omega, summ, seg_first, seg_count, pos, st)
                   : launch_build_f32<128, 4>(s, K, omega, summ, seg_first, seg_count, pos, st);
}
}  // namespace radar_impl

// The fused decode kernel (phi(q), scores, top-k, union, attention and merge
// of one (b, kv head) in R workgroups) and its select-only instantiation,
// for one feature count: this unit is compiled once per n with
// -DRADAR_FUSED_N=<n>, so the instantiations build in parallel.
#include "radar_impl.h"

#ifndef RADAR_FUSED_N
#error "compile with -DRADAR_FUSED_N=<feature count>"
#endif

namespace radar_impl {

// ---------------------------------------------------------------------------
// k_decode_fused: the whole decode step of one (b, kv head) in R workgroups
// ---------------------------------------------------------------------------
// Every workgroup of a pair runs the whole selection itself (phases 1-4 give
// the same result in each: the same inputs, the same order of operations),
// so no stage hands data to another workgroup (the per-XCD L2s are not
// coherent, so a cross-workgroup hand-off would need a kernel boundary or a
// cache flush). With R = 1 (at least as many pairs as compute units) one
// 512-thread workgroup per pair keeps every CU streaming and writes the
// output; with fewer pairs R workgroups share a pair's attention tiles and
// each writes a partial that k_combine merges (the repeated summary reads
// mostly hit the caches). Phases:
//   1. phi(q) of the group's G heads into LDS (16 lanes per Omega row;
//      Omega in fp32 or bf16, obf), with each wave's first summary rows
//      already in flight (waves whose first row is past the candidates
//      load none);
//   2. Eq. 6 scores of all candidates into LDS (16 or 32 summary rows per
//      wave per pass, streaming loads; above n = 512 each 16-row batch in
//      feature chunks, and phase 1 writes phi(q) to LDS chunk by chunk);
//   3. waves < G take the top-k of one head each, while the other waves
//      already attend the window tiles (the window never depends on the
//      selection);
//   4. the group's union in LDS;
//   5. every wave attends segment tiles (tile i to workgroup i mod R, and
//      in it to wave (i / R) mod 8);
//   6. the waves' online-softmax states merge in LDS into the output (or
//      the workgroup's partial).
// MODE kFusedSelect stops after phase 4 and writes the union to uni_out /
// ucnt_out for the split path's attention (the select path: one workgroup
// per pair replaces the phi(q), score and top-k kernels). MODE kFusedScored
// starts at phase 3: the scores of phases 1-2 come from the split path's
// chip-wide phi(q) and score kernels (gscores [nsl][B][Hq][nc_cap]), for pairs
// whose summary rows are too many to read R times (the scored path).

template <typename T, int D, int G, int N, int MODE>
__global__ __launch_bounds__(512) void k_decode_fused(
    const T* __restrict__ q, const T* __restrict__ K, const T* __restrict__ V,
    const void* __restrict__ omega, bool obf, const float* __restrict__ summ,
    T* __restrict__ out, int32_t* __restrict__ selected,
    float* __restrict__ sel_scores, int Hq, int Hkv, int64_t cap,
    int64_t s_cap, int tiles_per_seg, SeqArgs sa, int per_head, float s1,
    float s2, float inv_sqrt_n, float qscale, int* __restrict__ uni_out,
    int* __restrict__ ucnt_out, int umax, AppendArgs ap, int R, int n_pairs,
    float* __restrict__ part, int maxwg, const float* __restrict__ gscores,
    int nc_cap, int nsl, int64_t sl_stride, uint64_t* __restrict__ clk, int clk_max) {
  constexpr bool SEL = MODE == kFusedSelect;
  constexpr bool SCORED = MODE == kFusedScored;
  constexpr int NW = kFusedWaves;
  constexpr int FPL = N / 64;              // features per lane (phase 2)
  using TA = Tile<T, D, G>;
  // One LDS area serves the phases in turn: phi(q), the scores and the top-k
  // lists (dead after the top-k), the K rows of the waves' tiles, and the
  // waves' accumulators at the end. The waves that attend window tiles
  // beside the top-k are those >= G: their K rows lie past the first part
  // (at d = 64 with many features all K rows follow it).
  constexpr int SEL_BYTES = G * ((SCORED ? 0 : N) + kFusedMaxCand) * 4 + G * kMaxK * 8;
  constexpr int MRG_BYTES = NW * G * D * 4;
  constexpr int KROWS = SEL ? 0 : NW * TA::kLdsBytes;
  constexpr int KOFF = SEL_BYTES <= G * TA::kLdsBytes ? 0 : SEL_BYTES;
  constexpr int AREA = std::max({SEL_BYTES, SEL ? 0 : MRG_BYTES, KOFF + KROWS});
  static_assert(G <= (SCORED ? kScoredMaxG : kFusedMaxG), "group");
  static_assert(N % (4 * NW) == 0, "features");

  __shared__ __attribute__((aligned(16))) unsigned char area[AREA];
  __shared__ int sel_lds[G * kMaxK];
  __shared__ unsigned bits_lds[G * kBitmapWords];
  __shared__ int uni_lds[G * kMaxK];
  __shared__ float wm[NW][G], wl[NW][G];
  __shared__ int ucnt_lds;
  u64* list_lds = reinterpret_cast<u64*>(area);          // [G][kMaxK]
  float* phq = reinterpret_cast<float*>(area + G * kMaxK * 8);   // [G][N]
  float* sc = phq + (SCORED ? 0 : G * N);                // [G][kFusedMaxCand]
  float* wacc = reinterpret_cast<float*>(area);          // [NW][G][D]

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // measurement hook: the first thread stamps the phase boundaries (every
  // stamp starts as the entry time: phases 1-2 when they do not run keep it;
  // later stamps are written on every path)
  const bool clocked = clk != nullptr && (int)blockIdx.x < clk_max;   // uniform
  uint64_t* const cw = clk + (clocked ? (int64_t)blockIdx.x * RADAR_CLOCK_STAMPS : 0);
  auto stamp = [&](int i) {
    if (clocked && tid == 0) cw[i] = (uint64_t)wall_clock64();
  };
  if (clocked && tid == 0) {
    const uint64_t t0 = (uint64_t)wall_clock64();
#pragma unroll
    for (int i = 0; i < RADAR_CLOCK_STAMPS; ++i) cw[i] = t0;
  }
  // workgroup rj < R of pair bh: the workgroups of a pair differ by a
  // multiple of n_pairs, so they share an XCD (and its L2) when n_pairs is a
  // multiple of 8 (dealing a pair's workgroups over all XCDs instead measured
  // 2% slower on the scored path at 512K)
  // (the divisions run on the vector unit: readfirstlane keeps what follows
  // from them, loop counters and addresses, in scalar registers)
  const int rj = __builtin_amdgcn_readfirstlane((int)(blockIdx.x / (unsigned)n_pairs));
  const int pair = (int)blockIdx.x - rj * n_pairs;
  const int64_t bh = pair;
  const int64_t b = __builtin_amdgcn_readfirstlane(pair / Hkv);
  const int64_t hk = pair - b * Hkv;
  const T* q0 = q + (b * Hq + hk * G) * D;
  const Span sp = seq_span(sa, b);
  const int c = sa.c, k = sa.k, n_cand = sp.n_cand, k_eff = sp.k_eff;
  const int64_t ws = sp.ws, t = sp.t;

  // The append of radar_append_decode: the last wave writes the pair's new
  // row before anything reads it. The row belongs to the window (never to a
  // candidate segment), read from phase 3 on, after a barrier: those of
  // phases 1 and 2, or this one when there are no candidates (or no phases
  // 1 and 2).
  if (ap.K) {                              // uniform
    if (wave == NW - 1) append_row(ap, cap, bh, Hkv, lane);
    if (n_cand == 0 || SCORED) __syncthreads();
  }

  if constexpr (!SCORED) {
  if (n_cand > 0) {                        // uniform
    // Each wave's first batch of summary rows goes in flight before phi(q)
    // is computed (the rows do not depend on it), so the projection's
    // latency overlaps the stream of the scores.
    constexpr int RB = FPL <= 4 ? 2 : 1;   // 16-row batches per pass
    constexpr int FC = FPL < 4 ? FPL : 4;  // ... of a chunk
    const float* base = summ + (bh * s_cap) * N + lane * FC;
    // feature e of this lane's: four consecutive ones of each chunk of 256, so
    // that a load instruction reads whole lines (eight in a row, n = 512: half of
    // each line per instruction, 24.0 us a step instead of 20.8 for 32 pairs of
    // one head and 175 rows)
    auto at = [](int e) { return e / 4 * 256 + e % 4; };   // from base
    float x[RB][16][FPL];
    auto load_rows = [&](int rb) {
#pragma unroll
      for (int bt = 0; bt < RB; ++bt)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int row = min(rb + bt * 16 + i, n_cand - 1);
          const float* src = base + (int64_t)row * N;
          if constexpr (FPL % 4 == 0) {
#pragma unroll
            for (int e = 0; e < FPL; e += 4) {
              const float4 v = ld_stream_f4(src + at(e));
              x[bt][i][e] = v.x; x[bt][i][e + 1] = v.y;
              x[bt][i][e + 2] = v.z; x[bt][i][e + 3] = v.w;
            }
          } else if constexpr (FPL == 2) {
            const float2 v = *reinterpret_cast<const float2*>(src + at(0));
            x[bt][i][0] = v.x; x[bt][i][1] = v.y;
          } else {
            x[bt][i][0] = src[at(0)];
          }
        }
    };

    // ---- 1. phi(q) -----------------------------------------------------
    // 16 lanes per Omega row, 4 rows per wave and pass, NP passes in chunks.
    // The first chunk's Omega loads go out first, then q, then the summary rows
    // (when they fit in registers next to them). For bf16 caches the phase is
    // compiled once per Omega storage type and one copy runs, so all those
    // loads stay in flight together.
    const int rb0 = wave * 16 * RB;
    auto phase1 = [&](auto bf_tag) {
      constexpr bool BF = decltype(bf_tag)::value;
      constexpr int NP = N / (4 * NW);
      // (no summary rows are held beside them above n = 256)
      constexpr int PC = N > 256 && sizeof(T) == 2 ? 16 : (NP < 8 ? NP : 8);
      using PM = PhiRows<T, D, G, PC>;
      PM pm;
#pragma unroll
      for (int c0 = 0; c0 < NP; c0 += PC) {
        typename PM::template Om<BF> om;
        PM::template load<BF>(om, omega, c0 * 4 * NW + wave * 4 + (lane >> 4), 4 * NW, lane);
        if (c0 == 0) {
          pm.load_q(q0, lane);
          // rows clamp to the last candidate; a wave whose first row is
          // past it has no rows (the candidate count is uniform)
          if (N <= 256 && rb0 < n_cand) load_rows(rb0);
          pm.norm(s2, lane);
        }
        pm.template features<BF>(om, s1, inv_sqrt_n, lane, [&](int g, int p, float v) {
          phq[g * N + (c0 + p) * 4 * NW + wave * 4 + (lane >> 4)] = v;
        });
      }
      if (N == 512 && rb0 < n_cand) load_rows(rb0);
    };
    if constexpr (sizeof(T) == 2) {
      if (obf) phase1(std::true_type{});
      else phase1(std::false_type{});
    } else {
      phase1(std::false_type{});
    }
    __syncthreads();
    stamp(1);

    // ---- 2. scores ------------------------------------------------------
    // a chunk's sum of row (lane & 15) for one head (tree_add's order)
    auto dot = [&](const float* pq, auto&& row_at) -> float {
      float part[16];
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const float* xr = row_at(i);
        float a = 0.f;
#pragma unroll
        for (int e = 0; e < FC; ++e) a = fmaf(xr[e], pq[e], a);
        part[i] = a;
      }
      transpose_reduce<16>(part, lane);
      float v = part[0];
      v = xor_sum<16>(v);
      return xor_sum<32>(v);
    };
    if constexpr (N > 512) {
      // a 16-row batch's chunks one after another, the next one (of this batch
      // or the wave's next) requested before this one's products
      constexpr int NCH = FPL / 4;
      const float* rbase = summ + (bh * s_cap) * N + lane * 4;
      auto load_chunk = [&](float (&xx)[16][4], int rb, int ch) {
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int row = min(rb + i, n_cand - 1);
          const float4 f = ld_stream_f4(rbase + (int64_t)row * N + ch * 256);
          xx[i][0] = f.x; xx[i][1] = f.y; xx[i][2] = f.z; xx[i][3] = f.w;
        }
      };
      auto chunk_dot = [&](const float (&xx)[16][4], int ch, int g) {
        float pq[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) pq[e] = phq[g * N + ch * 256 + lane * 4 + e];
        return dot(pq, [&](int i) { return xx[i]; });
      };
      // few rows: S waves share a batch, each with a run of its chunks, and their
      // sums are added pairwise (8 candidates at n = 2048, four pairs of one head:
      // 16.8 us a step, 18.9 with a wave per batch; 192 pairs of four heads with
      // 10 candidates: 87.6 and 94.5)
      int S = 1;
      while (S * 4 <= NCH && (n_cand + 15) / 16 * (S * 2) <= NW) S *= 2;
      const int first = wave % S * (NCH / S), last = first + NCH / S;
      float xa[16][4], xb[16][4];
      int rb = wave / S * 16;
      if (rb < n_cand) load_chunk(xa, rb, first);
      for (; rb < n_cand; rb += NW * 16) {
        float hold[G][3], v[G];
#pragma unroll 1
        for (int ch = first; ch < last; ch += 2) {
          load_chunk(xb, rb, ch + 1);
          // (keeps the chunk's loads together and here: the compiler would sink
          // each to its first use and wait on one at a time)
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int g = 0; g < G; ++g) v[g] = chunk_dot(xa, ch, g);
          if (ch + 2 < last) load_chunk(xa, rb, ch + 2);
          else if (rb + NW * 16 < n_cand) load_chunk(xa, rb + NW * 16, 0);
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int g = 0; g < G; ++g)
            v[g] = tree_add(v[g] + chunk_dot(xb, ch + 1, g), (ch - first) / 2, hold[g]);
        }
        const int row = rb + (lane & 15);
#pragma unroll
        for (int g = 0; g < G; ++g)
          if (lane < 16 && row < n_cand) sc[g * kFusedMaxCand + wave % S * 64 + row] = v[g];
      }
      if (S > 1) {                         // uniform; at most 64 rows
        __syncthreads();
        float* mine = sc + wave * kFusedMaxCand + lane;
        if (wave < G && lane < n_cand) {
          float v = mine[0] + mine[64];
          if (S == 4) v += mine[128] + mine[192];
          mine[0] = v;
        }
      }
    } else {
      float pq[G][FPL];
#pragma unroll
      for (int g = 0; g < G; ++g)
#pragma unroll
        for (int e = 0; e < FPL; ++e) pq[g][e] = phq[g * N + lane * FC + at(e)];
      for (int rb = rb0; rb < n_cand; rb += NW * 16 * RB) {
        if (rb != rb0) load_rows(rb);
#pragma unroll
        for (int bt = 0; bt < RB; ++bt) {
          const int row = rb + bt * 16 + (lane & 15);
#pragma unroll
          for (int g = 0; g < G; ++g) {
            float v = dot(&pq[g][0], [&](int i) { return &x[bt][i][0]; });
            if constexpr (FPL == 8) v += dot(&pq[g][4], [&](int i) { return &x[bt][i][4]; });
            if (lane < 16 && row < n_cand) sc[g * kFusedMaxCand + row] = v;
          }
        }
      }
    }
    __syncthreads();
    stamp(2);
  }
  }

  // ---- 3. top-k (waves < G) | window and sink tiles (the other waves) ----
  // (a group of eight has no wave to spare: its window tiles come with the
  // segments' in phase 5)
  constexpr bool kBeside = G < NW;
  TA ta;
  if constexpr (!SEL) ta.init(q0, qscale, lane);
  unsigned char* const krows = area + KOFF + wave * TA::kLdsBytes;
  const int win_tiles = (int)((t - ws + kTile - 1) / kTile);
  const int extra_tiles = win_tiles + (sp.sink + kTile - 1) / kTile;
  auto extra_tile = [&](int i) {
    TileRef r;
    r.hmask = kAllHeads;
    if (i < win_tiles) {
      const int64_t start = ws + (int64_t)i * kTile;
      r.row0 = bh * cap + start;
      r.len = (int)min((int64_t)kTile, t - start);
    } else {
      const int off = (i - win_tiles) * kTile;
      r.row0 = bh * cap + off - sa.n_sink;
      r.len = min(kTile, sp.sink - off);
    }
    return r;
  };
  if (wave < G) {
    const int64_t hq = hk * G + wave;
    // every workgroup of the pair selects the same segments; the first
    // one reports them
    int32_t* so = selected && rj == 0 ? selected + (b * Hq + hq) * (int64_t)k : nullptr;
    float* sco = sel_scores && rj == 0 ? sel_scores + (b * Hq + hq) * (int64_t)k : nullptr;
    const float* src = SCORED ? gscores + (b * Hq + hq) * (int64_t)nc_cap
                              : sc + wave * kFusedMaxCand;
    if (SCORED && nsl > 1) {               // uniform; n_cand <= kFusedMaxCand
      add_slices(src, nsl, sl_stride, n_cand, sc + wave * kFusedMaxCand, lane);
      src = sc + wave * kFusedMaxCand;
    }
    int* row = sel_lds + wave * k_eff;
    u64* list = list_lds + wave * kMaxK;
    const int npl = (n_cand + 63) / 64;
    if (npl <= 1) head_topk<1>(src, n_cand, k, k_eff, row, so, sco, lane, list);
    else if (npl <= 2) head_topk<2>(src, n_cand, k, k_eff, row, so, sco, lane, list);
    else if (npl <= 4) head_topk<4>(src, n_cand, k, k_eff, row, so, sco, lane, list);
    else if (npl <= 8) head_topk<8>(src, n_cand, k, k_eff, row, so, sco, lane, list);
    else if (!SCORED || npl <= 16)
      head_topk<16>(src, n_cand, k, k_eff, row, so, sco, lane, list);
    else if constexpr (SCORED)             // up to 2048 candidates
      head_topk<32>(src, n_cand, k, k_eff, row, so, sco, lane, list);
  } else if constexpr (!SEL) {
    ta.run(K, V, rj + (wave - G) * R, extra_tiles, (NW - G) * R, krows, extra_tile);
  }
  __syncthreads();
  stamp(3);

  // ---- 4. union -----------------------------------------------------------
  // With one query head per group its selection is the set to attend (in
  // score order; the online softmax does not depend on the order), so the
  // bitmap union is skipped.
  const int* segs = sel_lds;
  int n_segs = k_eff;
  if constexpr (G > 1 || SEL) {
    group_union(sel_lds, bits_lds, G, k_eff, per_head != 0, uni_lds, &ucnt_lds);
    __syncthreads();
    segs = uni_lds;
    n_segs = ucnt_lds;
  }
  stamp(4);
  if constexpr (SEL) {                     // hand the union to the split path
    for (int i = tid; i < n_segs; i += NW * 64) uni_out[bh * umax + i] = segs[i];
    if (tid == 0) ucnt_out[bh] = n_segs;
    stamp(5);
    stamp(6);
    return;
  }
  const int seg_tiles = n_segs * tiles_per_seg;

  // ---- 5. segment tiles ---------------------------------------------------
  // (64-row tiles dealt round robin over the pair's waves; equal shares of
  // rows instead, cut at segment ends, measured slower: the shares start
  // mid-tile, so waves run more partial tiles, each costing nearly a whole
  // one)
  ta.run(K, V, rj + wave * R, seg_tiles + (kBeside ? 0 : extra_tiles), NW * R, krows, [&](int i) {
    if (!kBeside && i >= seg_tiles) return extra_tile(i - seg_tiles);
    const int e = segs[i / tiles_per_seg];
    const int s = e & ((1 << kUniIdBits) - 1);
    const int off = (i % tiles_per_seg) * kTile;
    // (the plain selection of a one-head group carries no head mask)
    return TileRef{bh * cap + (int64_t)s * c + off, min(kTile, c - off),
                   (G > 1 && per_head) ? (unsigned)e >> kUniIdBits : kAllHeads};
  });

  // ---- 6. merge -----------------------------------------------------------
  __syncthreads();                         // the K rows are dead from here on
  stamp(5);
  ta.finish(wacc + wave * G * D, wm[wave], wl[wave]);
  __syncthreads();
  for (int x = tid; x < G * D; x += NW * 64) {
    const int g = x / D, e = x % D;
    float M = wm[0][g];
#pragma unroll
    for (int w = 1; w < NW; ++w) M = fmaxf(M, wm[w][g]);
    float a = 0.f, L = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const float f = wm[w][g] == -INFINITY ? 0.f : fast_exp2(wm[w][g] - M);
      a = fmaf(wacc[(w * G + g) * D + e], f, a);
      L = fmaf(wl[w][g], f, L);
    }
    if (R == 1) {
      const float o = !sp.ok ? __uint_as_float(0x7fc00000u) : (L > 0.f ? a / L : 0.f);
      out[(b * Hq + hk * G + g) * D + e] = from_f32<T>(o);
    } else {                               // partial of this workgroup's tiles
      float* pj = part + ((bh * maxwg + rj) * G + g) * (int64_t)(D + 4);
      pj[4 + e] = a;
      if (e == 0) { pj[0] = M; pj[1] = L; }
    }
  }
  if (clocked) {
    __syncthreads();
    stamp(6);
  }
}

// The launch helpers below are compiled once per unit, each with its own
// RADAR_FUSED_N: internal linkage keeps the units' copies apart.
namespace {

template <typename T, int D, int G, int MODE>
radar_status launch_fused_tdg(const FusedArgs& a) {
  const Shape& s = *a.s;
  // the scored kernel reads no summaries: one instantiation serves every n
  constexpr int N = MODE == kFusedScored ? 64 : RADAR_FUSED_N;
  const float s1 = kLog2e / std::pow((float)s.d, 0.25f);
  const float s2 = kLog2e / (2.f * std::sqrt((float)s.d));
  const int n_pairs = s.B * s.Hkv;
  const int kind = MODE == kFusedSelect ? RADAR_K_SELECT
                   : MODE == kFusedScored ? RADAR_K_SCORED : RADAR_K_FUSED;
  launch(kind, k_decode_fused<T, D, G, N, MODE>,
         dim3((unsigned)(n_pairs * a.R)), dim3(kFusedWaves * 64), 0, a.st,
         reinterpret_cast<const T*>(a.q), reinterpret_cast<const T*>(a.K),
         reinterpret_cast<const T*>(a.V), a.omega, s.obf, a.summ,
         reinterpret_cast<T*>(a.out), a.selected, a.sel_scores, s.Hq, s.Hkv, s.cap,
         s.s_cap, (int)ceil_div(s.c, kTile), a.sa, s.per_head, s1, s2,
         1.f / std::sqrt((float)s.n), kLog2e / std::sqrt((float)s.d), a.uni_out,
         a.ucnt_out, a.umax, a.ap, a.R, n_pairs, a.part, a.maxwg, a.gscores, a.nc_cap,
         a.sp.nsl, a.sp.stride, g_clock, g_clock_max);
  return launch_status();
}

template <typename T, int D, int MODE>
radar_status launch_fused_td(const FusedArgs& a) {
  switch (a.s->G) {
    case 1: return launch_fused_tdg<T, D, 1, MODE>(a);
    case 2: return launch_fused_tdg<T, D, 2, MODE>(a);
    case 4: return launch_fused_tdg<T, D, 4, MODE>(a);
    default:
      if constexpr (MODE == kFusedScored && sizeof(T) == 2)
        return launch_fused_tdg<T, D, 8, MODE>(a);
      return RADAR_EUNSUPPORTED;
  }
}

// fp32 caches with d = 128 have no instantiation of the whole step (reading
// 16 KB of Omega per 32 features in every workgroup costs more than the two
// score kernels' launch): the host asks for their selection or scored modes
template <int MODE>
radar_status launch_fused_mode(const FusedArgs& a) {
  const Shape& s = *a.s;
  if (s.dt == RADAR_BF16)
    return s.d == 64 ? launch_fused_td<bf16_t, 64, MODE>(a) : launch_fused_td<bf16_t, 128, MODE>(a);
  if (s.d == 64) return launch_fused_td<float, 64, MODE>(a);
  if constexpr (MODE != kFusedFull) return launch_fused_td<float, 128, MODE>(a);
  return RADAR_EUNSUPPORTED;
}

}  // namespace

#define RADAR_FUSED_ENTRY2(n) launch_fused_n##n
#define RADAR_FUSED_ENTRY(n) RADAR_FUSED_ENTRY2(n)
radar_status RADAR_FUSED_ENTRY(RADAR_FUSED_N)(const FusedArgs& a, bool sel) {
  return sel ? launch_fused_mode<kFusedSelect>(a) : launch_fused_mode<kFusedFull>(a);
}

#if RADAR_FUSED_N == 64
radar_status launch_fused_scored(const FusedArgs& a) {
  return launch_fused_mode<kFusedScored>(a);
}
#endif

}  // namespace radar_impl

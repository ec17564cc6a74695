// The split decode path's stages, each spread over the whole chip: phi(q) and
// Eq. 6 scores, the exact segment mass, top-k and union, the given-selection
// union, the gather attention and the merge of its partials (also used by
// the fused path when several workgroups share a pair).
#include "radar_impl.h"

namespace radar_impl {

// ---------------------------------------------------------------------------
// k_phi_score: phi(q) (Eq. 4) and the segment scores a[h][s] = phi(q_h) .
// summ[s] (Eq. 6) in one kernel
// ---------------------------------------------------------------------------
// Grid (row blocks, pairs, feature slices). A workgroup computes phi(q) of its
// slice of fs features into LDS, with its first summary rows already in
// flight, and then scores 16 * NW rows of the slice, 16 per wave, in chunks of
// 64 * FPL features (each chunk of a row one contiguous wave load). A slice's scores go to their own array; the top-k adds the
// slices in order.
// Small calls are bound by latency: two kernels, with phi(q) through memory
// between them, took 11.5 us for the paper's 16K settings (8 pairs, 120 rows
// of 2048 features) where this one takes 7.5, and the step went from 32.9 to
// 30.2 us (80.0 to 78.7 us at 512K, 104 to 101 us for six ragged sequences with
// eight heads per group). Slices are what spreads few rows with many features
// over the chip without every workgroup reading all of Omega.
template <typename T, int D, int G, int FPL, int NW>
__global__ __launch_bounds__(64 * NW) void k_phi_score(
    const T* __restrict__ q, const void* __restrict__ omega, bool obf,
    const float* __restrict__ summ, float* __restrict__ scores, int Hq, int Hkv, int n, int fs,
    SeqArgs sa, int64_t s_cap, int nc_cap, int64_t sl_stride, float s1, float s2,
    float inv_sqrt_n) {
  constexpr int FC = 64 * FPL;             // features per chunk
  extern __shared__ __attribute__((aligned(16))) float phq[];   // [G][fs]
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t bh = blockIdx.y;
  const int64_t b = __builtin_amdgcn_readfirstlane((int)blockIdx.y / Hkv);
  const int64_t hk = bh - b * Hkv;
  const int n_cand = seq_span(sa, b).n_cand;
  if ((int)blockIdx.x * 16 * NW >= n_cand) return;     // workgroup-uniform
  const int f0 = blockIdx.z * fs;
  const T* q0 = q + (b * Hq + hk * G) * D;
  const float* base = summ + bh * s_cap * n + f0 + lane * FPL;

  float xa[16][FPL];
  // (an opaque row length: the sixteen addresses are worked out again for each
  // chunk; kept across chunks they took all registers and spilled, 45.8 us for
  // a step with four sequences of 1995 candidates at n = 512, 39.6 without. Not
  // for the first chunk, 0.2 us of a small call, nor where eight heads hold one)
  auto load_rows = [&](float (&x)[16][FPL], int row0, int ch) {
    int len = n;
    if (G <= 4 && ch > 0) asm volatile("" : "+s"(len));
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float* src = base + (int64_t)min(row0 + r, n_cand - 1) * len + ch * FC;
      if constexpr (FPL == 4) {
        const float4 v = ld_stream_f4(src);
        x[r][0] = v.x; x[r][1] = v.y; x[r][2] = v.z; x[r][3] = v.w;
      } else if constexpr (FPL == 2) {
        const float2 v = *reinterpret_cast<const float2*>(src);
        x[r][0] = v.x; x[r][1] = v.y;
      } else {
        x[r][0] = src[0];
      }
    }
  };

  const int row0 = (int)blockIdx.x * 16 * NW + wave * 16;
  // compiled once per Omega storage type, so that all loads before the first
  // product stay in flight together
  auto phi = [&](auto bf_tag) {
    constexpr bool BF = decltype(bf_tag)::value;
    // (fp32 words of eight heads: half the passes, for the registers)
    constexpr int kMost = sizeof(T) == 4 && G == 8 ? 4 : 8;
    constexpr int NP = FC / (4 * NW) < kMost ? FC / (4 * NW) : kMost;
    using PM = PhiRows<T, D, G, NP>;
    PM pm;
    for (int c0 = 0; c0 < fs; c0 += NP * 4 * NW) {
      typename PM::template Om<BF> om;
      const int mine = c0 + wave * 4 + (lane >> 4);
      PM::template load<BF>(om, omega, f0 + mine, 4 * NW, lane);
      if (c0 == 0) {
        pm.load_q(q0, lane);
        if (row0 < n_cand) load_rows(xa, row0, 0);
        pm.norm(s2, lane);
      }
      pm.template features<BF>(om, s1, inv_sqrt_n, lane, [&](int g, int p, float v) {
        phq[g * fs + mine + p * 4 * NW] = v;
      });
    }
  };
  if constexpr (sizeof(T) == 2) {
    if (obf) phi(std::true_type{});
    else phi(std::false_type{});
  } else {
    phi(std::false_type{});
  }
  __syncthreads();

  float* out = scores + blockIdx.z * sl_stride + (b * Hq + hk * G) * (int64_t)nc_cap;
  const int nch = fs / FC;                 // 1, 2, 4 or 8; 1 with FPL < 4
  if (row0 >= n_cand) return;              // wave-uniform, no barrier follows
  float hold[G][3];                        // chunk sums (tree_add)
  auto products = [&](const float (&x)[16][FPL], int ch) {
    float pq[G][FPL];
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
      for (int e = 0; e < FPL; ++e) pq[g][e] = phq[g * fs + ch * FC + lane * FPL + e];
    // keep the chunk's loads together (the compiler would otherwise sink
    // each to its first use and wait on one at a time)
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int g = 0; g < G; ++g) {
      float part[16];
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        float a = 0.f;
#pragma unroll
        for (int e = 0; e < FPL; ++e) a = fmaf(x[r][e], pq[g][e], a);
        part[r] = a;
      }
      transpose_reduce<16>(part, lane);
      float v = part[0];
      v = xor_sum<16>(v);
      v = xor_sum<32>(v);
      v = tree_add(v, ch, hold[g]);
      if (ch == nch - 1 && lane < 16 && row0 + lane < n_cand)
        out[g * (int64_t)nc_cap + row0 + lane] = v;
    }
  };
  // the next chunk's loads go out before this one's products where the
  // registers hold two (up to four heads); a single chunk, what small calls
  // take, by itself (before a loop the compiler works out every row's address:
  // 0.4 us of a step)
  if (FPL < 4 || nch == 1) {
    products(xa, 0);
    return;
  }
  if constexpr (FPL == 4 && G <= 4) {
    float xb[16][FPL];
#pragma unroll 1
    for (int ch = 0; ch < nch; ch += 2) {
      load_rows(xb, row0, ch + 1);
      products(xa, ch);
      if (ch + 2 < nch) load_rows(xa, row0, ch + 2);
      products(xb, ch + 1);
    }
  } else if constexpr (FPL == 4) {
#pragma unroll 1
    for (int ch = 0; ch < nch; ++ch) {
      if (ch > 0) load_rows(xa, row0, ch);
      products(xa, ch);
    }
  }
}

// ---------------------------------------------------------------------------
// k_phi, k_score: the same as two kernels (score_plan says when)
// ---------------------------------------------------------------------------
// k_phi: phi(q) of 64 features of one (b, kv head) per workgroup.
template <typename T, int D, int G, bool BF>
__global__ __launch_bounds__(256) void k_phi(const T* __restrict__ q,
                                             const void* __restrict__ omega,
                                             float* __restrict__ phiq, int n, int Hq, int Hkv,
                                             float s1, float s2, float inv_sqrt_n) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t bh = blockIdx.y;
  const int64_t hq0 = bh / Hkv * Hq + bh % Hkv * G;    // the group's first (b, q head)
  using PM = PhiRows<T, D, G, 4>;
  PM pm;
  typename PM::template Om<BF> om;
  const int row = blockIdx.x * 64 + wave * 4 + (lane >> 4);
  PM::template load<BF>(om, omega, row, 16, lane);
  pm.load_q(q + hq0 * D, lane);
  pm.norm(s2, lane);
  pm.template features<BF>(om, s1, inv_sqrt_n, lane, [&](int g, int p, float v) {
    phiq[(hq0 + g) * n + row + 16 * p] = v;
  });
}

// k_score: workgroup = 1, 2 or 4 waves x (16 * RB) summary rows of one (b, kv head)
// (fewer waves per workgroup when that spreads a small call over more CUs;
// the waves are independent). Lane l holds min(4, n / 64) features of phi(q)
// for the G heads of the group and a chunk of 256 features; each chunk of a
// row is one contiguous wave load, and all of a batch's rows are loaded before
// any is reduced. A 16-row batch is transpose-reduced inside each 16-lane row
// with DPP, then summed over the four rows.
// With S > 1 the S waves of a workgroup share one batch of rows instead and
// each takes two of the chunks (one round trip to memory instead of one per
// chunk or two for a wave that walks them all); the waves' row sums are added
// in LDS, pairwise.
template <int N, int G, int S>
__global__ __launch_bounds__(256) void k_score(const float* __restrict__ phiq,
                                               const float* __restrict__ summ,
                                               float* __restrict__ scores,
                                               int Hq, int Hkv, SeqArgs sa,
                                               int64_t s_cap, int nc_cap) {
  constexpr int FC = N < 256 ? N / 64 : 4; // features per lane and chunk
  constexpr int NCH = N / (64 * FC);       // chunks (1 for n <= 256)
  constexpr int RB = N <= 256 ? 2 : 1;     // 16-row batches per wave
  constexpr int CPW = NCH / S;             // chunks of each wave
  static_assert(CPW * S == NCH && CPW <= 2 && (S == 1 || RB == 1), "feature split");
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int64_t bh = blockIdx.y;
  const int64_t b = bh / Hkv, hk = bh % Hkv;
  const int n_cand = seq_span(sa, b).n_cand;
  const int wrow0 = S > 1 ? blockIdx.x * 16
                          : (blockIdx.x * (blockDim.x >> 6) + wave) * (16 * RB);
  // wave-uniform, and workgroup-uniform with S > 1 (the waves share rows),
  // so the barrier below is reached by all waves or by none
  if (wrow0 >= n_cand) return;
  const int ch0 = S > 1 ? wave * CPW : 0;  // this wave's first chunk

  // chunk ch holds features ch * 64 * FC + lane * FC + e (e < FC) of lane
  // `lane`, so each chunk of a row is one contiguous 64 * FC * 4-byte load
  const float* base = summ + (bh * s_cap) * N + lane * FC;
  // a chunk's phi(q) features and rows
  auto load_chunk = [&](int ch, float (&pq)[G][FC], float (&x)[RB][16][FC]) {
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const float* src = phiq + ((b * Hq + hk * G + g) * N) + ch * 64 * FC + lane * FC;
#pragma unroll
      for (int e = 0; e < FC; ++e) pq[g][e] = src[e];
    }
#pragma unroll
    for (int bt = 0; bt < RB; ++bt)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int row = min(wrow0 + bt * 16 + r, n_cand - 1);
        const float* src = base + (int64_t)row * N + ch * 64 * FC;
        if constexpr (FC == 4) {
          const float4 v = ld_stream_f4(src);
          x[bt][r][0] = v.x; x[bt][r][1] = v.y; x[bt][r][2] = v.z; x[bt][r][3] = v.w;
        } else if constexpr (FC == 2) {
          const float2 v = *reinterpret_cast<const float2*>(src);
          x[bt][r][0] = v.x; x[bt][r][1] = v.y;
        } else {
          x[bt][r][0] = src[0];
        }
      }
  };
  // the chunk's sum of row (lane & 15) for one head
  auto dot = [&](const float (&pq)[FC], const float (&x)[16][FC]) -> float {
    float part[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      float a = 0.f;
#pragma unroll
      for (int e = 0; e < FC; ++e) a = fmaf(x[r][e], pq[e], a);
      part[r] = a;
    }
    transpose_reduce<16>(part, lane);
    float v = part[0];
    v = xor_sum<16>(v);
    return xor_sum<32>(v);
  };
  float sum[RB][G];
  // Of two chunks both are in flight before the first products up to four heads
  // (eight would not fit).
  if constexpr (CPW == 2 && G <= 4) {
    float pqa[G][FC], xa[RB][16][FC], pqb[G][FC], xb[RB][16][FC];
    load_chunk(ch0, pqa, xa);
    load_chunk(ch0 + 1, pqb, xb);
    // (the compiler would otherwise sink each load to its first use and wait
    // on one load at a time)
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int g = 0; g < G; ++g) sum[0][g] = dot(pqa[g], xa[0]);
#pragma unroll
    for (int g = 0; g < G; ++g) sum[0][g] += dot(pqb[g], xb[0]);
  } else {
#pragma unroll 1
    for (int ch = 0; ch < CPW; ++ch) {
      float pq[G][FC], x[RB][16][FC];
      load_chunk(ch0 + ch, pq, x);
      if constexpr (CPW > 1) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int bt = 0; bt < RB; ++bt)
#pragma unroll
        for (int g = 0; g < G; ++g) {
          const float v = dot(pq[g], x[bt]);
          sum[bt][g] = ch > 0 ? sum[bt][g] + v : v;
        }
    }
  }
  if constexpr (S > 1) {
    __shared__ float red[S][G][16];
    if (lane < 16) {
#pragma unroll
      for (int g = 0; g < G; ++g) red[wave][g][lane] = sum[0][g];
    }
    __syncthreads();
    if (wave == 0 && lane < 16 && wrow0 + lane < n_cand) {
#pragma unroll
      for (int g = 0; g < G; ++g) {
        float v = red[0][g][lane] + red[1][g][lane];
        if constexpr (S == 4) v += red[2][g][lane] + red[3][g][lane];
        scores[(b * Hq + hk * G + g) * (int64_t)nc_cap + wrow0 + lane] = v;
      }
    }
  } else {
#pragma unroll
    for (int bt = 0; bt < RB; ++bt) {
      const int row = wrow0 + bt * 16 + lane;
      if (lane < 16 && row < n_cand) {
#pragma unroll
        for (int g = 0; g < G; ++g)
          scores[(b * Hq + hk * G + g) * (int64_t)nc_cap + row] = sum[bt][g];
      }
    }
  }
}

// ---------------------------------------------------------------------------
// k_topk_union: top-k of every query head, union per kv head
// ---------------------------------------------------------------------------
// One workgroup per (b, kv head); wave w takes heads w, w + 4, ... of the
// group. The heads' sorted selections go to LDS and the union of the group
// (ascending ids) to the workspace for the attention stage.
__global__ __launch_bounds__(256) void k_topk_union(
    const float* __restrict__ scores, int nsl, int64_t sl_stride, int Hq, int Hkv, int G,
    SeqArgs sa, int nc_cap, int per_head, int* __restrict__ uni, int* __restrict__ ucnt,
    int umax, int32_t* __restrict__ selected, float* __restrict__ sel_scores,
    AppendArgs ap, int64_t cap) {
  __shared__ int sel_lds[kMaxG * kMaxK];
  __shared__ unsigned bits_lds[kMaxG * kBitmapWords];
  __shared__ u64 list_lds[4][kMaxK];
  __shared__ float sum_lds[4][kFusedMaxCand];
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int64_t bh = blockIdx.x;
  const int64_t b = bh / Hkv, hk = bh % Hkv;
  // the append of radar_append_decode (the attention kernel that reads the
  // row runs after this one)
  if (ap.K && wave == 3) append_row(ap, cap, bh, Hkv, lane);
  const Span sp = seq_span(sa, b);
  const int n_cand = sp.n_cand, k_eff = sp.k_eff, k = sa.k;
  const int npl = (n_cand + 63) / 64;
  u64* list = list_lds[wave];
  for (int hl = wave; hl < G; hl += 4) {
    const int64_t hq = hk * G + hl;
    const float* src = scores + (b * Hq + hq) * (int64_t)nc_cap;
    if (nsl > 1) {                         // uniform; n_cand <= kFusedMaxCand
      add_slices(src, nsl, sl_stride, n_cand, sum_lds[wave], lane);
      src = sum_lds[wave];
    }
    int32_t* so = selected ? selected + (b * Hq + hq) * (int64_t)k : nullptr;
    float* sco = sel_scores ? sel_scores + (b * Hq + hq) * (int64_t)k : nullptr;
    int* row = sel_lds + hl * k_eff;
    if (npl <= 1) head_topk<1>(src, n_cand, k, k_eff, row, so, sco, lane, list);
    else if (npl <= 2) head_topk<2>(src, n_cand, k, k_eff, row, so, sco, lane, list);
    else if (npl <= 4) head_topk<4>(src, n_cand, k, k_eff, row, so, sco, lane, list);
    else if (npl <= 8) head_topk<8>(src, n_cand, k, k_eff, row, so, sco, lane, list);
    else if (npl <= 16) head_topk<16>(src, n_cand, k, k_eff, row, so, sco, lane, list);
    else head_topk<32>(src, n_cand, k, k_eff, row, so, sco, lane, list);
  }
  __syncthreads();
  group_union(sel_lds, bits_lds, G, k_eff, per_head != 0, uni + bh * umax,
              ucnt + bh);
}


// ---------------------------------------------------------------------------
// k_segment_mass: exact segment attention mass, ln(beta_s) per query head
// ---------------------------------------------------------------------------
// beta_s = sum over the keys of segment s of exp(q . k / sqrt(d)) (the
// segment's unnormalised attention weight; selecting its top-k is the exact
// segment search). One wave per candidate segment: the logits of each
// <= 64-token tile come from the same row-contiguous loads and
// transpose-reduce as the attention tiles, and an online log-sum-exp in
// base 2 carries across the segment's tiles. Writes ln(beta_s) to
// scores[b][h][s].
template <typename T, int D, int G>
__global__ __launch_bounds__(256) void k_segment_mass(
    const T* __restrict__ q, const T* __restrict__ K, float* __restrict__ scores,
    int Hq, int Hkv, int64_t cap, SeqArgs sa, int nc_cap, float qscale, int with_rest) {
  constexpr int EPL = Elem<T>::kPer16;
  constexpr int LPR = D / EPL;
  constexpr int RPI = kWave / LPR;
  constexpr int ITER = kTile / RPI;
  constexpr float kLn2 = 0.69314718055994530942f;
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int64_t bh = blockIdx.y;
  const int64_t b = bh / Hkv, hk = bh % Hkv;
  const int c = sa.c;
  const int s = blockIdx.x * 4 + wave;
  const Span sp = seq_span(sa, b);
  // item n_cand (with_rest): the tokens in no candidate segment, the window
  // and the sinks, whose mass every selection keeps
  if (s > sp.n_cand || (s == sp.n_cand && !with_rest)) return;  // wave-uniform
  const int r = lane / LPR, jj = lane % LPR;

  float qf[G][EPL];
#pragma unroll
  for (int g = 0; g < G; ++g) {
    const uint4 u = *reinterpret_cast<const uint4*>(
        q + ((b * Hq + hk * G + g) * D + jj * EPL));
    unpack16<T>(u, qf[g]);
#pragma unroll
    for (int e = 0; e < EPL; ++e) qf[g][e] *= qscale;
  }
  float m[G], l[G];
#pragma unroll
  for (int g = 0; g < G; ++g) { m[g] = -INFINITY; l[g] = 0.f; }

  // rows [row0, row0 + len) after the pair's base, 1 <= len <= 64: an
  // online log-sum-exp in base 2 across the tiles
  auto tile = [&](int64_t row0, int len) {
    const T* kbase = K + (bh * cap + row0) * D + jj * EPL;
    uint4 kr[ITER];
#pragma unroll
    for (int i = 0; i < ITER; ++i)
      kr[i] = ld_stream(kbase + (int64_t)min(i * RPI + r, len - 1) * D);
    float pl[G][ITER];
#pragma unroll
    for (int i = 0; i < ITER; ++i) {
      float kf[EPL];
      unpack16<T>(kr[i], kf);
#pragma unroll
      for (int g = 0; g < G; ++g) {
        float a = 0.f;
#pragma unroll
        for (int e = 0; e < EPL; ++e) a = fmaf(qf[g][e], kf[e], a);
        pl[g][i] = a;
      }
    }
    const bool mine_ok = (jj * RPI + r) < len;
#pragma unroll
    for (int g = 0; g < G; ++g) {
      transpose_reduce<LPR>(pl[g], lane);
      const float lg = pl[g][0];
      const float mt = wave_max(mine_ok ? lg : -INFINITY);
      const float mn = fmaxf(m[g], mt);
      const float p = mine_ok ? fast_exp2(lg - mn) : 0.f;
      l[g] = fmaf(l[g], fast_exp2(m[g] - mn), wave_sum(p));
      m[g] = mn;
    }
  };
  if (s < sp.n_cand) {
    for (int off = 0; off < c; off += kTile) tile((int64_t)s * c + off, min(kTile, c - off));
  } else {
    for (int64_t st = sp.ws; st < sp.t; st += kTile) tile(st, (int)min((int64_t)kTile, sp.t - st));
    for (int off = 0; off < sp.sink; off += kTile)
      tile((int64_t)off - sa.n_sink, min(kTile, sp.sink - off));
  }
  if (lane == 0) {
#pragma unroll
    for (int g = 0; g < G; ++g)
      scores[(b * Hq + hk * G + g) * (int64_t)nc_cap + s] =
          l[g] > 0.f ? (m[g] + __log2f(l[g])) * kLn2 : -INFINITY;
  }
}


// ---------------------------------------------------------------------------
// k_union_given: union of caller-given selections (attention on a supplied
// selection, the last step of Algorithm 1 alone)
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_union_given(
    const int32_t* __restrict__ given, int given_k, int Hq, int Hkv, int G,
    SeqArgs sa, int per_head, int* __restrict__ uni, int* __restrict__ ucnt,
    int umax) {
  __shared__ int sel_lds[kMaxG * kMaxK];
  __shared__ unsigned bits_lds[kMaxG * kBitmapWords];
  const int64_t bh = blockIdx.x;
  const int64_t b = bh / Hkv, hk = bh % Hkv;
  const int n_cand = seq_span(sa, b).n_cand;
  const int M = G * given_k;
  for (int i = threadIdx.x; i < M; i += 256) {
    const int hl = i / given_k, r = i % given_k;
    const int id = given[(b * Hq + hk * G + hl) * (int64_t)given_k + r];
    sel_lds[i] = (id >= 0 && id < n_cand) ? id : -1;
  }
  __syncthreads();
  group_union(sel_lds, bits_lds, G, given_k, per_head != 0, uni + bh * umax,
              ucnt + bh);
}


// ---------------------------------------------------------------------------
// k_attend: split attention, one partial (max, sum, acc[d]) per workgroup
// ---------------------------------------------------------------------------
// Tiles of a (b, kv head): tiles_per_seg per union segment, then ceil(|W| /
// 64) window tiles, then ceil(sinks / 64) sink tiles. Workgroup j takes
// tiles [4 tpw j, 4 tpw (j + 1)); wave w takes every fourth of them from
// 4 tpw j + w, with an online softmax across its tiles, and the workgroup
// merges its four waves in LDS. With per_head set, a segment tile counts
// only for the heads that selected the segment.
template <typename T, int D, int G>
__global__ __launch_bounds__(256) void k_attend(
    const T* __restrict__ q, const T* __restrict__ K, const T* __restrict__ V,
    const int* __restrict__ uni, const int* __restrict__ ucnt,
    float* __restrict__ part, int Hq, int Hkv, int64_t cap,
    int tiles_per_seg, SeqArgs sa, int per_head, int umax, int maxwg, int tpw,
    float qscale) {
  using TA = AttendTile<T, D, G>;
  constexpr int PSTRIDE = D + 4;
  constexpr int kMerge = 4 * G * D * 4;
  constexpr int kLds = 4 * TA::kLdsBytes > kMerge ? 4 * TA::kLdsBytes : kMerge;

  __shared__ float wm[4][G], wl[4][G];
  // the waves' K rows, then (when every wave is done) their accumulators
  __shared__ __attribute__((aligned(16))) unsigned char lds[kLds];
  float (*wacc)[G][D] = reinterpret_cast<float (*)[G][D]>(lds);

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t bh = blockIdx.y;
  const int64_t b = bh / Hkv, hk = bh % Hkv;
  const int j = blockIdx.x;
  const Span sp = seq_span(sa, b);
  const int c = sa.c;

  const int U = ucnt[bh];
  const int seg_tiles = U * tiles_per_seg;
  const int win_tiles = (int)(((int64_t)sp.t - sp.ws + kTile - 1) / kTile);
  const int total = seg_tiles + win_tiles + (sp.sink + kTile - 1) / kTile;
  const int nwg = (total + 4 * tpw - 1) / (4 * tpw);
  if (j >= nwg) return;

  TA ta;
  ta.init(q + (b * Hq + hk * G) * D, qscale, lane);
  const int t_end = min(total, (j + 1) * 4 * tpw);
  ta.run(K, V, j * 4 * tpw + wave, t_end, 4, lds + wave * TA::kLdsBytes, [&](int ti) {
    TileRef r;
    r.hmask = kAllHeads;
    if (ti < seg_tiles) {
      const int e = uni[bh * umax + ti / tiles_per_seg];
      const int s = e & ((1 << kUniIdBits) - 1);
      if (per_head) r.hmask = (unsigned)e >> kUniIdBits;
      const int off = (ti % tiles_per_seg) * kTile;
      r.row0 = bh * cap + (int64_t)s * c + off;
      r.len = min(kTile, c - off);
    } else if (ti < seg_tiles + win_tiles) {
      const int64_t start = sp.ws + (int64_t)(ti - seg_tiles) * kTile;
      r.row0 = bh * cap + start;
      r.len = (int)min((int64_t)kTile, sp.t - start);
    } else {
      const int off = (ti - seg_tiles - win_tiles) * kTile;
      r.row0 = bh * cap + off - sa.n_sink;
      r.len = min(kTile, sp.sink - off);
    }
    return r;
  });
  __syncthreads();                         // no wave reads its K rows any more
  ta.finish(&wacc[wave][0][0], wm[wave], wl[wave]);
  __syncthreads();

  float* pj = part + ((bh * maxwg + j) * G) * (int64_t)PSTRIDE;
  for (int x = tid; x < G * D; x += 256) {
    const int g = x / D, e = x % D;
    float M = wm[0][g];
#pragma unroll
    for (int w = 1; w < 4; ++w) M = fmaxf(M, wm[w][g]);
    float a = 0.f, L = 0.f;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const float f = wm[w][g] == -INFINITY ? 0.f : fast_exp2(wm[w][g] - M);
      a = fmaf(wacc[w][g][e], f, a);
      L = fmaf(wl[w][g], f, L);
    }
    pj[g * PSTRIDE + 4 + e] = a;
    if (e == 0) { pj[g * PSTRIDE] = M; pj[g * PSTRIDE + 1] = L; }
  }
}

// ---------------------------------------------------------------------------
// k_combine: log-sum-exp merge of the partials of each (b, q head)
// ---------------------------------------------------------------------------
// Grid (B * Hq, D / DS), NT threads: each workgroup produces DS output dims
// of one query head from at most MAXP partials. Every workgroup takes the
// maximum and the scaled sum over all the head's partials (a (max, sum)
// pair each, kept in registers between the passes); then the NT / DS groups
// of threads sum disjoint subsets of the partials' accumulators over its
// dims, and LDS adds the groups.
// With many partials per head (DS = 32, MAXP = kMaxWg) a head's partials are
// read by several CUs at once, and each thread issues its first PF
// accumulator loads before the first reduction, so most of the merge waits
// on memory once. With few (DS = D, PF = 0) one workgroup per head saves the
// launches, and the accumulators are read after the reductions.
template <typename T, int D, int NT, int DS, int MAXP, int PF>
__global__ __launch_bounds__(NT) void k_combine(
    const float* __restrict__ part, const int* __restrict__ ucnt,
    T* __restrict__ out, int Hq, int Hkv, int G, int tiles_per_seg,
    SeqArgs sa, int maxwg, int tpw, int fixed_nwg) {
  constexpr int PSTRIDE = D + 4;
  constexpr int NWAVE = NT / kWave;
  constexpr int NGRP = NT / DS;            // thread groups over the partials
  constexpr int PPT = (MAXP + NT - 1) / NT;  // (max, sum) pairs per thread
  static_assert(D % DS == 0 && MAXP <= kMaxWg && PF * NGRP <= MAXP, "shape");
  __shared__ float f_lds[MAXP];
  __shared__ float red_lds[2 * NWAVE];
  __shared__ float acc_lds[NT];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t bhq = blockIdx.x;
  const int e0 = blockIdx.y * DS;
  const int64_t b = bhq / Hq, hq = bhq % Hq;
  const int64_t hk = hq / G;
  const int g = (int)(hq % G);
  const int64_t bh = b * Hkv + hk;
  const Span sp = seq_span(sa, b);
  // partials of the pair: fixed_nwg (one per workgroup of the fused
  // kernel), or one per 4 tpw tiles of the split attention; the host sizes
  // MAXP from the same bound
  int nwg = fixed_nwg;
  if (nwg == 0) {
    const int extra = (int)(((int64_t)sp.t - sp.ws + kTile - 1) / kTile) +
                      (sp.sink + kTile - 1) / kTile;
    nwg = (ucnt[bh] * tiles_per_seg + extra + 4 * tpw - 1) / (4 * tpw);
  }
  nwg = min(nwg, MAXP);
  T* o = out + bhq * D + e0;
  if (!sp.ok || nwg == 0) {                // invalid length / nothing attended
    if (tid < DS) o[tid] = from_f32<T>(sp.ok ? 0.f : __uint_as_float(0x7fc00000u));
    return;
  }
  const float* pb = part + ((bh * maxwg) * G + g) * (int64_t)PSTRIDE;
  const int64_t wstride = (int64_t)G * PSTRIDE;

  float mw[PPT], lw[PPT];
#pragma unroll
  for (int i = 0; i < PPT; ++i) {
    const int w = tid + i * NT;
    mw[i] = w < nwg ? pb[w * wstride] : -INFINITY;
    lw[i] = w < nwg ? pb[w * wstride + 1] : 0.f;
  }
  const int e = tid % DS, grp = tid / DS;
  const float* pe = pb + 4 + e0 + e;
  float av[PF > 0 ? PF : 1];
#pragma unroll
  for (int j = 0; j < PF; ++j) {
    const int w = grp + j * NGRP;
    av[j] = w < nwg ? pe[w * wstride] : 0.f;
  }

  float mx = -INFINITY;
#pragma unroll
  for (int i = 0; i < PPT; ++i) mx = fmaxf(mx, mw[i]);
  mx = wave_max(mx);
  if (lane == 0) red_lds[wave] = mx;
  __syncthreads();
  float M = red_lds[0];
#pragma unroll
  for (int i = 1; i < NWAVE; ++i) M = fmaxf(M, red_lds[i]);
  if (M == -INFINITY) {                    // this head attended nothing
    if (tid < DS) o[tid] = from_f32<T>(0.f);
    return;
  }
  float ls = 0.f;
#pragma unroll
  for (int i = 0; i < PPT; ++i) {
    const int w = tid + i * NT;
    if (w < nwg) {
      const float f = fast_exp2(mw[i] - M);
      f_lds[w] = f;
      ls = fmaf(lw[i], f, ls);
    }
  }
  ls = wave_sum(ls);
  if (lane == 0) red_lds[NWAVE + wave] = ls;
  __syncthreads();
  float L = 0.f;
#pragma unroll
  for (int i = 0; i < NWAVE; ++i) L += red_lds[NWAVE + i];
  float a = 0.f;
#pragma unroll
  for (int j = 0; j < PF; ++j) {
    const int w = grp + j * NGRP;
    if (w < nwg) a = fmaf(av[j], f_lds[w], a);
  }
#pragma unroll 8
  for (int w = grp + PF * NGRP; w < nwg; w += NGRP) a = fmaf(pe[w * wstride], f_lds[w], a);
  acc_lds[tid] = a;
  __syncthreads();
  if (tid < DS) {
    float sum = 0.f;
#pragma unroll
    for (int i = 0; i < NGRP; ++i) sum += acc_lds[i * DS + tid];
    o[tid] = from_f32<T>(sum / L);
  }
}

// ---- decode pieces -------------------------------------------------------
// n_cand: the largest candidate count of the call (grid size); each
// workgroup reads its sequence's own from sa
template <int N, int G>
void launch_score_ng(const Shape& s, const float* phiq, const float* summ,
                     float* scores, int n_cand, const SeqArgs& sa, hipStream_t st) {
  // above n = 512 the waves of a workgroup split a batch's chunks, two each
  constexpr int S = N > 512 ? N / 512 : 1;
  if constexpr (S > 1) {
    const dim3 grid((unsigned)ceil_div(n_cand, 16), (unsigned)(s.B * s.Hkv));
    const int nc_cap = (int)std::max<int64_t>(1, s.s_cap);
    launch(RADAR_K_SCORE, k_score<N, G, S>, grid, dim3(64 * S), 0, st, phiq, summ, scores,
           s.Hq, s.Hkv, sa, s.s_cap, nc_cap);
  } else {
    constexpr int rows_per_wave = 16 * (N <= 256 ? 2 : 1);
    // waves per workgroup: 4 when that still gives two workgroups per CU,
    // else fewer, so that the rows spread over more CUs (n = 512, where the
    // slices of few pairs had no room; large tables always give them)
    int wpb = 4;
    while (wpb > 1 && ceil_div(n_cand, rows_per_wave * wpb) * s.B * s.Hkv < 2 * num_cu())
      wpb >>= 1;
    const dim3 grid((unsigned)ceil_div(n_cand, rows_per_wave * wpb), (unsigned)(s.B * s.Hkv));
    const int nc_cap = (int)std::max<int64_t>(1, s.s_cap);
    launch(RADAR_K_SCORE, k_score<N, G, 1>, grid, dim3(64 * wpb), 0, st, phiq, summ, scores,
           s.Hq, s.Hkv, sa, s.s_cap, nc_cap);
  }
}

template <int N>
void launch_score_n(const Shape& s, const float* phiq, const float* summ,
                    float* scores, int n_cand, const SeqArgs& sa, hipStream_t st) {
  switch (s.G) {
    case 1: launch_score_ng<N, 1>(s, phiq, summ, scores, n_cand, sa, st); break;
    case 2: launch_score_ng<N, 2>(s, phiq, summ, scores, n_cand, sa, st); break;
    case 4: launch_score_ng<N, 4>(s, phiq, summ, scores, n_cand, sa, st); break;
    default: launch_score_ng<N, 8>(s, phiq, summ, scores, n_cand, sa, st); break;
  }
}

void launch_score(const Shape& s, const float* phiq, const float* summ,
                  float* scores, int n_cand, const SeqArgs& sa, hipStream_t st) {
  switch (s.n) {
    case 64: launch_score_n<64>(s, phiq, summ, scores, n_cand, sa, st); break;
    case 128: launch_score_n<128>(s, phiq, summ, scores, n_cand, sa, st); break;
    case 256: launch_score_n<256>(s, phiq, summ, scores, n_cand, sa, st); break;
    case 512: launch_score_n<512>(s, phiq, summ, scores, n_cand, sa, st); break;
    case 1024: launch_score_n<1024>(s, phiq, summ, scores, n_cand, sa, st); break;
    default: launch_score_n<2048>(s, phiq, summ, scores, n_cand, sa, st); break;
  }
}

// Feature slices of k_phi_score: one, doubled (down to 256 features each)
// while the call has fewer workgroups than CUs. Where the slices would not fit
// (their scores in the workspace's array of n + capacity / c floats per query
// head, a head's sums in LDS), k_phi and k_score, whose waves split the
// features within a workgroup (1180 rows x 2048 features, six pairs of four
// heads: 40.6 us a step, 52.3 with one slice; 871 x 1024, eight pairs: 36.2 and
// 38.6; 512 features: 29-38 us, up to 10% less than with one slice).
// Large summary tables (from 64 MB) take k_phi and k_score: streaming is all
// there is to them then, and k_score's many small workgroups balance better
// (56 pairs x 1302 rows x 2048 features, four heads: 161 us a step, 183 with
// k_phi_score; 8 x 120 x 2048: 32.9 and 30.2).
ScorePlan score_plan(const Shape& s, int n_cand) {
  const int64_t cap = std::max<int64_t>(1, s.s_cap);
  const int64_t stride = (int64_t)s.B * s.Hq * cap;
  if ((int64_t)n_cand * s.n * 4 * s.B * s.Hkv >= (64 << 20)) return {0, 0};
  const int64_t rows = std::max<int64_t>(1, ceil_div(n_cand, 128)) * s.B * s.Hkv;
  int nsl = 1;
  while (s.n / nsl > 256 && rows * nsl < num_cu()) nsl *= 2;
  if (nsl > 1 && (n_cand > kFusedMaxCand || nsl * cap > s.n + cap)) return {0, 0};
  return {nsl, stride};
}

template <typename T, int D, int G>
void launch_phi_score(const Shape& s, const void* q, const void* omega, const float* summ,
                      float* sc, int n_cand, const ScorePlan& sp, const SeqArgs& sa,
                      hipStream_t st) {
  const float s1 = kLog2e / std::pow((float)s.d, 0.25f);
  const float s2 = kLog2e / (2.f * std::sqrt((float)s.d));
  const int fs = s.n / sp.nsl, P = s.B * s.Hkv;
  // four waves per workgroup where eight would leave CUs idle
  const bool narrow = ceil_div(n_cand, 128) * P * sp.nsl < num_cu();
  const dim3 grid((unsigned)ceil_div(n_cand, narrow ? 64 : 128), (unsigned)P, (unsigned)sp.nsl);
  auto go = [&](auto fpl, auto nw) {
    constexpr int NW = decltype(nw)::value;
    launch(RADAR_K_SCORE, k_phi_score<T, D, G, decltype(fpl)::value, NW>, grid, dim3(64 * NW),
           (size_t)G * fs * 4, st, static_cast<const T*>(q), omega, s.obf, summ, sc, s.Hq,
           s.Hkv, s.n, fs, sa, s.s_cap, (int)std::max<int64_t>(1, s.s_cap), sp.stride, s1, s2,
           1.f / std::sqrt((float)s.n));
  };
  auto go_nw = [&](auto fpl) {
    if (narrow) go(fpl, std::integral_constant<int, 4>{});
    else go(fpl, std::integral_constant<int, 8>{});
  };
  if (fs >= 256) go_nw(std::integral_constant<int, 4>{});
  else if (fs == 128) go_nw(std::integral_constant<int, 2>{});
  else go_nw(std::integral_constant<int, 1>{});
}

template <typename T, int D, int G>
void launch_phi(const Shape& s, const void* q, const void* omega, float* phiq, hipStream_t st) {
  const float s1 = kLog2e / std::pow((float)s.d, 0.25f);
  const float s2 = kLog2e / (2.f * std::sqrt((float)s.d));
  const dim3 grid((unsigned)(s.n / 64), (unsigned)(s.B * s.Hkv));
  auto go = [&](auto bf) {
    launch(RADAR_K_PHI_Q, k_phi<T, D, G, decltype(bf)::value>, grid, dim3(256), 0, st,
           static_cast<const T*>(q), omega, phiq, s.n, s.Hq, s.Hkv, s1, s2,
           1.f / std::sqrt((float)s.n));
  };
  if constexpr (sizeof(T) == 2) {
    if (s.obf) return go(std::true_type{});
  }
  go(std::false_type{});
}

void launch_scores(const Shape& s, const void* q, const void* omega, const float* summ,
                   float* base, int n_cand, const ScorePlan& sp, const SeqArgs& sa,
                   hipStream_t st) {
  float* sc = scores_of(s, base, sp);
  auto go_t = [&](auto tag, auto g) {
    typedef decltype(tag) T;
    constexpr int G = decltype(g)::value;
    if (sp.nsl == 0) {
      if (s.d == 64) launch_phi<T, 64, G>(s, q, omega, base, st);
      else launch_phi<T, 128, G>(s, q, omega, base, st);
      launch_score(s, base, summ, sc, n_cand, sa, st);
    } else {
      if (s.d == 64) launch_phi_score<T, 64, G>(s, q, omega, summ, sc, n_cand, sp, sa, st);
      else launch_phi_score<T, 128, G>(s, q, omega, summ, sc, n_cand, sp, sa, st);
    }
  };
  auto go = [&](auto g) {
    if (s.dt == RADAR_BF16) go_t(bf16_t{}, g);
    else go_t(float{}, g);
  };
  switch (s.G) {
    case 1: go(std::integral_constant<int, 1>{}); break;
    case 2: go(std::integral_constant<int, 2>{}); break;
    case 4: go(std::integral_constant<int, 4>{}); break;
    default: go(std::integral_constant<int, 8>{}); break;
  }
}

// The merge of the partials into the output: fixed_nwg partials per pair
// (the fused kernel's workgroups), or those of the split attention (tpw);
// partials_per_head bounds their count (at most kMaxWg). Above 128 the dims
// are split over D / 32 workgroups per head; otherwise one 256-thread
// workgroup per head (1024 threads measured the same or up to 0.5 us slower).
template <typename T, int D>
void launch_combine(const Shape& s, const float* part, const int* ucnt, void* out,
                    const SeqArgs& sa, const WsLayout& L, int tpw, int fixed_nwg,
                    int partials_per_head, hipStream_t st) {
  if (partials_per_head > 128)
    launch(RADAR_K_COMBINE, k_combine<T, D, 1024, 32, kMaxWg, 16>,
           dim3((unsigned)(s.B * s.Hq), (unsigned)(D / 32)), dim3(1024), 0, st, part,
           ucnt, reinterpret_cast<T*>(out), s.Hq, s.Hkv, s.G, L.tiles_per_seg, sa,
           L.maxwg, tpw, fixed_nwg);
  else
    launch(RADAR_K_COMBINE, k_combine<T, D, 256, D, 128, 0>, dim3((unsigned)(s.B * s.Hq)),
           dim3(256), 0, st, part, ucnt, reinterpret_cast<T*>(out), s.Hq, s.Hkv, s.G,
           L.tiles_per_seg, sa, L.maxwg, tpw, fixed_nwg);
}

template <typename T, int D, int G>
void launch_attend_g(const Shape& s, const void* q, const void* K, const void* V,
                     unsigned char* w, const WsLayout& L, int grid_x, int tpw,
                     const SeqArgs& sa, hipStream_t st) {
  const float qscale = kLog2e / std::sqrt((float)s.d);
  launch(RADAR_K_ATTEND, k_attend<T, D, G>,
         dim3((unsigned)grid_x, (unsigned)(s.B * s.Hkv)), dim3(256), 0, st,
         reinterpret_cast<const T*>(q), reinterpret_cast<const T*>(K),
         reinterpret_cast<const T*>(V), reinterpret_cast<const int*>(w + L.uni),
         reinterpret_cast<const int*>(w + L.ucnt), reinterpret_cast<float*>(w + L.part),
         s.Hq, s.Hkv, s.cap, L.tiles_per_seg, sa, s.per_head, L.umax, L.maxwg, tpw,
         qscale);
}

template <typename T, int D>
void launch_attend_d(const Shape& s, const void* q, const void* K, const void* V,
                     unsigned char* w, const WsLayout& L, int grid_x, int tpw,
                     const SeqArgs& sa, void* out, hipStream_t st) {
  switch (s.G) {
    case 1: launch_attend_g<T, D, 1>(s, q, K, V, w, L, grid_x, tpw, sa, st); break;
    case 2: launch_attend_g<T, D, 2>(s, q, K, V, w, L, grid_x, tpw, sa, st); break;
    case 4: launch_attend_g<T, D, 4>(s, q, K, V, w, L, grid_x, tpw, sa, st); break;
    default: launch_attend_g<T, D, 8>(s, q, K, V, w, L, grid_x, tpw, sa, st); break;
  }
  launch_combine<T, D>(s, reinterpret_cast<const float*>(w + L.part),
                       reinterpret_cast<const int*>(w + L.ucnt), out, sa, L, tpw, 0,
                       grid_x, st);
}

// Tiles beyond the union's segments per (b, kv head), the window's and the
// sinks': exact for one shared length, an upper bound over lengths in
// [1, t_max] for per-sequence lengths (a window never exceeds w + c - 1
// tokens nor the tokens after the sinks).
int64_t extra_tiles(const Shape& s, const SeqArgs& sa) {
  const Span sp = make_span(sa.t_max, sa);
  const int64_t win = sa.lens ? std::min<int64_t>(sp.t, (int64_t)s.w + s.c - 1)
                              : sp.t - sp.ws;
  return ceil_div(win, kTile) + ceil_div(sp.sink, kTile);
}

// Split of the attention work: tiles per wave (tpw) so that the grid still
// holds about eight workgroups per CU (a grid only just above the resident
// count leaves a long tail), but no more (fewer, larger workgroups mean fewer
// partials to merge); and the grid width per (b, kv head) for the largest
// union, at most the kMaxWg partials that a merge takes: a pair with more
// tiles gives its waves more of them.
AttendGrid attend_grid(const Shape& s, const WsLayout& L, int u_bound,
                       int64_t extra) {
  const int64_t per_bh = (int64_t)u_bound * L.tiles_per_seg + extra;
  const int64_t tiles = per_bh * s.B * s.Hkv;
  const int64_t tpw =
      std::max(std::min<int64_t>(8, std::max<int64_t>(1, tiles / (4 * 8 * num_cu()))),
               ceil_div(per_bh, 4 * kMaxWg));
  return {(int)ceil_div(per_bh, 4 * tpw), (int)tpw};
}

// exact attention over the union in the workspace, then the merge; K and V
// start after the sinks
radar_status launch_attend(const Shape& s, const void* q, const void* K,
                           const void* V, const AttendGrid& ag, const SeqArgs& sa,
                           void* out, unsigned char* w, const WsLayout& L,
                           hipStream_t st) {
  if (s.dt == RADAR_BF16) {
    if (s.d == 64) launch_attend_d<bf16_t, 64>(s, q, K, V, w, L, ag.grid_x, ag.tpw, sa, out, st);
    else launch_attend_d<bf16_t, 128>(s, q, K, V, w, L, ag.grid_x, ag.tpw, sa, out, st);
  } else {
    if (s.d == 64) launch_attend_d<float, 64>(s, q, K, V, w, L, ag.grid_x, ag.tpw, sa, out, st);
    else launch_attend_d<float, 128>(s, q, K, V, w, L, ag.grid_x, ag.tpw, sa, out, st);
  }
  return launch_status();
}

// ---- exact segment search ---------------------------------------------------
template <typename T, int D>
void launch_segment_mass_d(const Shape& s, const void* q, const void* K, float* scores,
                           int n_cand, const SeqArgs& sa, int nc_cap, bool with_rest,
                           hipStream_t st) {
  const int items = n_cand + (with_rest ? 1 : 0);
  const dim3 grid((unsigned)ceil_div(items, 4), (unsigned)(s.B * s.Hkv));
  const float qscale = kLog2e / std::sqrt((float)s.d);
  const T* qt = reinterpret_cast<const T*>(q);
  const T* Kt = reinterpret_cast<const T*>(K);
  const int wr = with_rest ? 1 : 0;
  switch (s.G) {
    case 1: launch(RADAR_K_SCORE, k_segment_mass<T, D, 1>, grid, dim3(256), 0, st, qt, Kt, scores, s.Hq, s.Hkv, s.cap, sa, nc_cap, qscale, wr); break;
    case 2: launch(RADAR_K_SCORE, k_segment_mass<T, D, 2>, grid, dim3(256), 0, st, qt, Kt, scores, s.Hq, s.Hkv, s.cap, sa, nc_cap, qscale, wr); break;
    case 4: launch(RADAR_K_SCORE, k_segment_mass<T, D, 4>, grid, dim3(256), 0, st, qt, Kt, scores, s.Hq, s.Hkv, s.cap, sa, nc_cap, qscale, wr); break;
    default: launch(RADAR_K_SCORE, k_segment_mass<T, D, 8>, grid, dim3(256), 0, st, qt, Kt, scores, s.Hq, s.Hkv, s.cap, sa, nc_cap, qscale, wr); break;
  }
}
// ---- entry points for the other units ---------------------------------------
void launch_segment_mass(const Shape& s, const void* q, const void* K, float* scores,
                         int n_cand, const SeqArgs& sa, int nc_cap, bool with_rest,
                         hipStream_t st) {
  if (s.dt == RADAR_BF16) {
    if (s.d == 64) launch_segment_mass_d<bf16_t, 64>(s, q, K, scores, n_cand, sa, nc_cap, with_rest, st);
    else launch_segment_mass_d<bf16_t, 128>(s, q, K, scores, n_cand, sa, nc_cap, with_rest, st);
  } else {
    if (s.d == 64) launch_segment_mass_d<float, 64>(s, q, K, scores, n_cand, sa, nc_cap, with_rest, st);
    else launch_segment_mass_d<float, 128>(s, q, K, scores, n_cand, sa, nc_cap, with_rest, st);
  }
}

void launch_topk_union(const Shape& s, const float* scores, const ScorePlan& sp,
                       const SeqArgs& sa, int* uni, int* ucnt, int umax, int32_t* selected,
                       float* sel_scores, const AppendArgs& ap, hipStream_t st) {
  launch(RADAR_K_TOPK, k_topk_union, dim3((unsigned)(s.B * s.Hkv)), dim3(256), 0, st,
         scores, sp.nsl, sp.stride, s.Hq, s.Hkv, s.G, sa, (int)std::max<int64_t>(1, s.s_cap),
         s.per_head,
         uni, ucnt, umax, selected, sel_scores, ap, s.cap);
}

void launch_union_given(const Shape& s, const int32_t* given, int given_k,
                        const SeqArgs& sa, int* uni, int* ucnt, int umax,
                        hipStream_t st) {
  launch(RADAR_K_TOPK, k_union_given, dim3((unsigned)(s.B * s.Hkv)), dim3(256), 0, st,
         given, given_k, s.Hq, s.Hkv, s.G, sa, s.per_head, uni, ucnt, umax);
}

void launch_combine_any(const Shape& s, const float* part, const int* ucnt, void* out,
                        const SeqArgs& sa, const WsLayout& L, int tpw, int fixed_nwg,
                        int partials_per_head, hipStream_t st) {
  if (s.dt == RADAR_BF16) {
    if (s.d == 64)
      launch_combine<bf16_t, 64>(s, part, ucnt, out, sa, L, tpw, fixed_nwg, partials_per_head, st);
    else
      launch_combine<bf16_t, 128>(s, part, ucnt, out, sa, L, tpw, fixed_nwg, partials_per_head, st);
  } else {
    if (s.d == 64)
      launch_combine<float, 64>(s, part, ucnt, out, sa, L, tpw, fixed_nwg, partials_per_head, st);
    else
      launch_combine<float, 128>(s, part, ucnt, out, sa, L, tpw, fixed_nwg, partials_per_head, st);
  }
}

}  // namespace radar_impl

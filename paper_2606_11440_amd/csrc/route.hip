// Route step of the tick: feature gather, policy MLP on MFMA, masked argmax.
//
// Sec. 3 Eq. 1 (the executor's state), Sec. 3 "Action" (a -> model a / K,
// depth a % K) and Sec. 4.2 (a policy network scores every joint action; it
// is deployed greedily here). A wave owns 32 or 64 request rows of the persistent
// kernels; in the feature-split kernels a block owns the rows and each wave some
// of every hidden layer's features.
//
// The MLP is evaluated transposed, Y^T = W X^T, on 32x32 MFMA tiles: the
// weights are the A operand (from LDS or L2, pre-packed so that each lane
// reads 16 contiguous bytes per instruction) and the activations are the B
// operand. The accumulator layout of one layer (lane = row n + 32 g, register v
// holds output feature 8(v/4) + 4g + v%4 of its tile) is used directly as the
// B operand of the next layer; the next layer's weight columns are permuted at
// pool creation to match, so a wave's activations never leave registers (the
// feature-split kernels hand them to the other waves through LDS).
//
// bf16 pools use v_mfma_f32_32x32x16_bf16 (fp32 accumulate, hidden activations
// rounded to bf16 after the ReLU); fp32 pools use v_mfma_f32_16x16x4_f32 on
// 16-row tiles in the same transposed scheme.
#include "route_dev.h"
#include "route_split.h"

namespace im {
namespace {

// ---------------------------------------------------------------------------
// fp32 policies on v_mfma_f32_16x16x4_f32, one wave per 16 rows (a light
// fp32 tick, ~16 K requests, still gives every SIMD a wave).
//
// Transposed form Y^T = W X^T: lane l serves row n = l % 16 of the wave's
// rows and K group q = l / 16. An output tile's accumulator holds features
// 16 T + 4 q + r (r = 0..3) of the lane's row: exactly the B operand of the
// next layer's K step (T, r), whose weight columns are permuted to match at
// pool creation, so activations never leave registers. Weights are packed so
// that one 16-byte load per lane covers four consecutive K steps; the hidden
// layers' loads run D steps ahead of their MFMAs.
// ---------------------------------------------------------------------------

// Masked argmax over the four lanes of a row (q = 0..3), action and logits
// stores, or the RL-rollout outputs; lane (n, q) holds actions 16 T + 4 q + r.
// Same rules as the 32-row epilogue: lowest action on exact ties, Philox block
// (id, env, action / 4) per four consecutive actions.
template <int AT>
__device__ __forceinline__ void epilogue16(const RowCtx& c, const f32x4 (&acc)[AT], int q) {
  const KernArgs a = late_args();
  // bit 16 T + r: action 16 T + 4 q + r is masked
  const uint64_t inv = (uint64_t)((int64_t)~c.amask >> (4 * q));
  const uint32_t mw[2] = {(uint32_t)inv, (uint32_t)(inv >> 32)};
  float zm[AT][4];
  const uint32_t low = minus_inf();
  float best = __uint_as_float(low);
#pragma unroll
  for (int T = 0; T < AT; ++T) {
#pragma unroll
    for (int r = 0; r < 4; ++r) zm[T][r] = mask_logit(acc[T][r], bit_ones(mw[T >> 1], 16 * (T & 1) + r), low);
    best = maximum3(best, zm[T][0], zm[T][1]);
    best = maximum3(best, zm[T][2], zm[T][3]);
  }
#pragma unroll
  for (int off = 16; off <= 32; off *= 2) {
    const float o = __shfl_xor(best, off, 64);
    best = maximum3(best, o, o);
  }
  // some row has a NaN among its valid logits (rare): best is kept NaN where the
  // lowest valid action's is, and is the largest of the others elsewhere
  if (ballot(best != best) != 0) {
    const int first = __ffsll((unsigned long long)c.amask) - 1 - 4 * q;
    float b = __uint_as_float(low);
    int32_t first_nan = 0;
#pragma unroll
    for (int T = 0; T < AT; ++T)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        b = max3(b, zm[T][r], zm[T][r]);
        first_nan |= first == 16 * T + r && zm[T][r] != zm[T][r];
      }
#pragma unroll
    for (int off = 16; off <= 32; off *= 2) {
      const float o = __shfl_xor(b, off, 64);
      b = max3(b, o, o);
      first_nan |= __shfl_xor(first_nan, off, 64);
    }
    if (!first_nan) best = b;
  }
  int32_t ba = 127;
#pragma unroll
  for (int T = AT - 1; T >= 0; --T)
#pragma unroll
    for (int r = 3; r >= 0; --r) ba = zm[T][r] == best ? 16 * T + r : ba;
  ba += 4 * q;
#pragma unroll
  for (int off = 16; off <= 32; off *= 2) ba = min(ba, __shfl_xor(ba, off, 64));
  ba = argmax_of(ba, c.amask, best);
  if (a->rl) {
    const bool sample = a->greedy == 0;
    uint32_t id = 0;
    if (sample) id = request_id(a, c);
    RlSums s;
    float val = 0.f;
#pragma unroll
    for (int T = 0; T < AT; ++T) {
      const float z[4] = {acc[T][0], acc[T][1], acc[T][2], acc[T][3]};
      const uint32_t mb = mw[T >> 1] >> (16 * (T & 1));
      if (16 * T < a->A) {   // uniform
        if (sample) {
          const uint4 w = philox10(make_uint4(id, (uint32_t)c.e, (uint32_t)(4 * T + q), 0u), a->seed_lo, a->seed_hi);
          rl_block<true>(s, z, mb, best, 16 * T + 4 * q, w);
        } else {
          rl_block<false>(s, z, mb, best, 16 * T + 4 * q, make_uint4(0, 0, 0, 0));
        }
      }
      if (a->value && (a->A >> 4) == T) {   // uniform: the tile of row A
        const int i = a->A & 3;
        const float v = i == 0 ? z[0] : (i == 1 ? z[1] : (i == 2 ? z[2] : z[3]));
        val = ((a->A >> 2) & 3) == q ? v : 0.f;
      }
    }
#pragma unroll
    for (int off = 16; off <= 32; off *= 2) {
      rl_join(s, __shfl_xor(s.s, off, 64), __shfl_xor(s.sz, off, 64), __shfl_xor(s.bs, off, 64),
              __shfl_xor(s.bz, off, 64), __shfl_xor(s.ba, off, 64));
      val += __shfl_xor(val, off, 64);             // one lane of the row holds row A
    }
    if (c.live && q == 0) rl_store(a, c, s, best, ba, val);
  } else if (c.live && q == 0) {
    a->actions[c.r] = c.bad ? -1 : ba;
    if (c.bad) atomicOr(a->err, c.bad);
  }
  if (!c.live) return;
  if (a->logits) {
    float* out = a->logits + (size_t)c.r * a->A;
#pragma unroll
    for (int T = 0; T < AT; ++T)
      store_logits(a, out, 16 * T + 4 * q, c.bad ? 0.f : acc[T][0], c.bad ? 0.f : acc[T][1], c.bad ? 0.f : acc[T][2],
                   c.bad ? 0.f : acc[T][3]);
  }
}

// One hidden-input layer: out[To] = bias + W h over K = 4 KG steps, the
// weights of step group (To, g) at W[(To KG + g) 64 + lane] (4 floats, one
// per K step of the group). With one wave per SIMD the MFMAs are ordered so
// that consecutive ones never share an accumulator: four output tiles at a
// time (weights of D groups in flight), or, for fewer than four tiles, each
// tile's K steps split over four partial sums added at the end.
template <int TO, int KG, int D>
__device__ __forceinline__ void layer16(const f32x4* W, const float* bias, const f32x4 (&h)[KG], int lane,
                                        int q, f32x4 (&out)[TO]) {
  if constexpr (TO % 4 == 0) {
    constexpr int N = (TO / 4) * KG;   // (tile quad, group) steps
    constexpr int DD = D < N ? D : N;
    f32x4 wr[DD][4];
    auto load = [&](int s, f32x4 (&w)[4]) {
      const int T4 = s / KG, g = s % KG;
#pragma unroll
      for (int t = 0; t < 4; ++t) w[t] = W[((4 * T4 + t) * KG + g) * 64 + lane];
    };
#pragma unroll
    for (int s = 0; s < DD; ++s) load(s, wr[s]);
#pragma unroll
    for (int T4 = 0; T4 < TO / 4; ++T4) {
      f32x4 acc[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) acc[t] = *(const f32x4*)(bias + ((4 * T4 + t) * 4 + q) * 4);
#pragma unroll
      for (int g = 0; g < KG; ++g) {
        const int st = T4 * KG + g;
        f32x4 w[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) w[t] = wr[st % DD][t];
        if (st + DD < N) load(st + DD, wr[st % DD]);
#pragma unroll
        for (int t = 0; t < 4; ++t) acc[t] = mfma16_f32(w[t].x, h[g].x, acc[t]);
#pragma unroll
        for (int t = 0; t < 4; ++t) acc[t] = mfma16_f32(w[t].y, h[g].y, acc[t]);
#pragma unroll
        for (int t = 0; t < 4; ++t) acc[t] = mfma16_f32(w[t].z, h[g].z, acc[t]);
#pragma unroll
        for (int t = 0; t < 4; ++t) acc[t] = mfma16_f32(w[t].w, h[g].w, acc[t]);
      }
#pragma unroll
      for (int t = 0; t < 4; ++t) out[4 * T4 + t] = acc[t];
    }
  } else {
    constexpr int N = TO * KG;
    constexpr int DD = 4 * D < N ? 4 * D : N;
    f32x4 wr[DD];
#pragma unroll
    for (int t = 0; t < DD; ++t) wr[t] = W[t * 64 + lane];
#pragma unroll
    for (int To = 0; To < TO; ++To) {
      f32x4 p[4];
      p[0] = *(const f32x4*)(bias + (To * 4 + q) * 4);
      p[1] = p[2] = p[3] = f32x4{};
#pragma unroll
      for (int g = 0; g < KG; ++g) {
        const int t = To * KG + g;
        const f32x4 w = wr[t % DD];
        if (t + DD < N) wr[t % DD] = W[(t + DD) * 64 + lane];
        p[0] = mfma16_f32(w.x, h[g].x, p[0]);
        p[1] = mfma16_f32(w.y, h[g].y, p[1]);
        p[2] = mfma16_f32(w.z, h[g].z, p[2]);
        p[3] = mfma16_f32(w.w, h[g].w, p[3]);
      }
      out[To] = (p[0] + p[1]) + (p[2] + p[3]);
    }
  }
}

// Features 16 g + 4 q .. + 3 of a row, the four K steps of group g in lane group
// q (fp32 pools): one 16-byte load of the embedding or of the env's load
// statistics where the embedding width is a multiple of 4.
__device__ __forceinline__ f32x4 feats16(const RouteArgs& a, const RowCtx& c, int g, int q) {
  const int k = 16 * g + 4 * q;
  const float* emb = (const float*)a.emb + (size_t)c.q * a.embed_dim;
  if ((a.embed_dim & 3) == 0) {
    const int k2 = k - a.embed_dim;   // 4 M is a multiple of 4 too: the four are of one kind
    if (k2 < 0) {
      const f32x4u v = *(const f32x4u*)(emb + k);   // the table itself may be only 4-byte aligned
      return (f32x4){v.x, v.y, v.z, v.w};
    }
    if (k2 < 4 * a.M) return *(const f32x4*)(a.snap + (size_t)c.e * snap_stride(a.M) + k2);
    f32x4 x = {};
    if (k2 == 4 * a.M) x.x = (float)c.budget * a.inv_bud;
    return x;
  }
  f32x4 x;
#pragma unroll
  for (int j = 0; j < 4; ++j) x[j] = k + j < a.embed_dim ? emb[k + j] : tail_feature(a, c, k + j);
  return x;
}

template <int H, int NL, int AT>
__global__ __launch_bounds__(256) void route_f32(RouteArgs a_in) {
  // chain pools: the tick's row count is on the device
  RouteArgs a = a_in;
  if (a_in.n_total_dev) a.n_total = min(*a_in.n_total_dev, a_in.n_total);   // the caller's buffers bound it
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int n = lane & 15, q = lane >> 4;
  const int32_t row0 = (int32_t)(blockIdx.x * 4 + wave) * 16;
  if (row0 >= a.n_total) return;
  const int32_t rl = row0 + 15 < a.n_total ? row0 + 15 : a.n_total - 1;
  const int32_t rows[1] = {row0 + n};
  const int32_t rsel[1] = {rows[0] < a.n_total ? rows[0] : a.n_total - 1};
  int32_t envs[1];
  find_envs<1>(a, row0, rl, rsel, envs);
  const RowCtx c = row_setup_env(a, rows[0], envs[0]);
  constexpr int TH = H / 16;   // hidden output tiles
  constexpr int KGH = H / 16;  // K step groups over a hidden layer (4 steps of 4 features)
  const f32x4* W1 = (const f32x4*)a.W[0];
  // layer 1: the K steps of group g carry features 16 g + 4 q .. + 3 in lane group q
  const int KG1 = (a.k1 + 3) / 4;
  f32x4 h1[TH];
#pragma unroll
  for (int T = 0; T < TH; ++T) h1[T] = *(const f32x4*)(a.bias[0] + (T * 4 + q) * 4);
  auto feats = [&](int g) { return feats16(a, c, g, q); };
  f32x4 x = feats(0);
  f32x4 wn[TH];
#pragma unroll
  for (int T = 0; T < TH; ++T) wn[T] = W1[(T * KG1) * 64 + lane];
  for (int g = 0; g < KG1; ++g) {
    f32x4 wc[TH];
#pragma unroll
    for (int T = 0; T < TH; ++T) wc[T] = wn[T];
    const f32x4 xc = x;
    if (g + 1 < KG1) {
      x = feats(g + 1);
#pragma unroll
      for (int T = 0; T < TH; ++T) wn[T] = W1[(T * KG1 + g + 1) * 64 + lane];
    }
    // K step by K step across the output tiles: consecutive MFMAs never
    // share an accumulator
#pragma unroll
    for (int T = 0; T < TH; ++T) h1[T] = mfma16_f32(wc[T].x, xc.x, h1[T]);
#pragma unroll
    for (int T = 0; T < TH; ++T) h1[T] = mfma16_f32(wc[T].y, xc.y, h1[T]);
#pragma unroll
    for (int T = 0; T < TH; ++T) h1[T] = mfma16_f32(wc[T].z, xc.z, h1[T]);
#pragma unroll
    for (int T = 0; T < TH; ++T) h1[T] = mfma16_f32(wc[T].w, xc.w, h1[T]);
  }
#pragma unroll
  for (int T = 0; T < TH; ++T)
#pragma unroll
    for (int r = 0; r < 4; ++r) h1[T][r] = relu(h1[T][r]);
  f32x4 out[AT];
  if constexpr (NL == 2) {
    layer16<AT, KGH, 2>((const f32x4*)a.W[1], a.bias[1], h1, lane, q, out);
  } else {
    f32x4 h2[TH];
    layer16<TH, KGH, 2>((const f32x4*)a.W[1], a.bias[1], h1, lane, q, h2);
#pragma unroll
    for (int T = 0; T < TH; ++T)
#pragma unroll
      for (int r = 0; r < 4; ++r) h2[T][r] = relu(h2[T][r]);
    layer16<AT, KGH, 2>((const f32x4*)a.W[2], a.bias[2], h2, lane, q, out);
  }
  epilogue16<AT>(c, out, q);
}

// TQ output tiles [To0, To0 + TQ) of a layer for NR row tiles over KG groups of
// inputs in LDS (`hs`: group g's 16-byte words of row tile j at
// hs[(g NR + j) 64 + lane]) while the weights (W[(To stride + g) 64 + lane],
// 4 floats) come through the caches D groups ahead. acc[t][j][0] holds the
// bias; NP partial sums per tile where too few tiles would otherwise share an
// accumulator between consecutive MFMAs.
template <int TQ, int NR, int NP, int D>
__device__ __forceinline__ void layer16_lds(const f32x4* W, int stride, int KG, const f32x4* hs, int To0, int lane,
                                            f32x4 (&acc)[TQ][NR][NP]) {
  const f32x4* Wl = W + (size_t)To0 * stride * 64 + lane;
  f32x4 wr[D][TQ];
#pragma unroll
  for (int d = 0; d < D; ++d)
#pragma unroll
    for (int t = 0; t < TQ; ++t) wr[d][t] = Wl[(t * stride + (d < KG ? d : KG - 1)) * 64];
  for (int g0 = 0; g0 < KG; g0 += D) {
#pragma unroll
    for (int d = 0; d < D; ++d) {
      const int g = g0 + d;
      if (g < KG) {
        f32x4 b[NR], w[TQ];
#pragma unroll
        for (int j = 0; j < NR; ++j) b[j] = hs[(g * NR + j) * 64 + lane];
        const int gn = g + D < KG ? g + D : KG - 1;
#pragma unroll
        for (int t = 0; t < TQ; ++t) {
          w[t] = wr[d][t];
          wr[d][t] = Wl[(t * stride + gn) * 64];
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int t = 0; t < TQ; ++t)
#pragma unroll
            for (int j = 0; j < NR; ++j) acc[t][j][i % NP] = mfma16_f32(w[t][i], b[j][i], acc[t][j][i % NP]);
      }
    }
  }
}

// The output layer of one row tile: its input groups are NR apart in LDS.
template <int AT, int NR, int NP, int D>
__device__ __forceinline__ void layer16_out(const f32x4* W, int KG, const f32x4* hs, int lane, f32x4 (&acc)[AT][1][NP]) {
  f32x4 wr[D][AT];
#pragma unroll
  for (int d = 0; d < D; ++d)
#pragma unroll
    for (int t = 0; t < AT; ++t) wr[d][t] = W[(t * KG + (d < KG ? d : KG - 1)) * 64 + lane];
  for (int g0 = 0; g0 < KG; g0 += D) {   // KG is a multiple of 4
#pragma unroll
    for (int d = 0; d < D; ++d) {
      const int g = g0 + d;
      const f32x4 b = hs[g * NR * 64 + lane];
      const int gn = g + D < KG ? g + D : KG - 1;
#pragma unroll
      for (int t = 0; t < AT; ++t) {
        const f32x4 w = wr[d][t];
        wr[d][t] = W[(t * KG + gn) * 64 + lane];
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[t][0][i % NP] = mfma16_f32(w[i], b[i], acc[t][0][i % NP]);
      }
    }
  }
}

// fp32 policies with hidden widths in whole tile quads, feature-split: one
// block of 4 waves per 16 NR rows, wave w computing output tiles
// [w TH/4, (w + 1) TH/4) of each hidden layer; the block exchanges features and
// activations through LDS (one buffer, rewritten layer by layer), and wave j
// computes the output layer and the epilogue of row tile j. The features come
// in once per block, a group (four K steps) per wave in turn.
template <int H>
constexpr int kF32Groups = H / 16 < 8 ? 8 : H / 16;   // groups of features in LDS at a time
template <int H, int NL, int AT, int NR>
__device__ __forceinline__ void f32s_block(const RouteArgs& a, int32_t row0, f32x4* hs) {
  constexpr int TH = H / 16, TQ = TH / 4, KGH = H / 16, ROWS = 16 * NR;
  constexpr int KC = kF32Groups<H>;
  constexpr int NP = TQ >= 4 ? 1 : 4;        // partial sums of the hidden layers after the first
  constexpr int NPO = AT >= 4 ? 1 : 4;       // of the output layer
  static_assert(TH % 4 == 0, "hidden tiles split four ways");
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n = lane & 15, q = lane >> 4;
  if (row0 >= a.n_total) return;   // the whole block (chain pools' bound launch)
  const int T0 = wave * TQ;
  const int KG1 = (a.k1 + 3) / 4;
  f32x4 bias1[TQ];
#pragma unroll
  for (int t = 0; t < TQ; ++t) bias1[t] = *(const f32x4*)(a.bias[0] + ((T0 + t) * 4 + q) * 4);
  const int32_t rlast = min(row0 + ROWS - 1, a.n_total - 1);
  int32_t rows[NR], rsel[NR], envs[NR];
#pragma unroll
  for (int j = 0; j < NR; ++j) {
    rows[j] = row0 + 16 * j + n;
    rsel[j] = min(rows[j], rlast);
  }
  find_envs<NR>(a, row0, rlast, rsel, envs);
  RowCtx c[NR];
#pragma unroll
  for (int j = 0; j < NR; ++j) c[j] = row_setup_env(a, rows[j], envs[j]);

  f32x4 h[TQ][NR][1];
#pragma unroll
  for (int t = 0; t < TQ; ++t)
#pragma unroll
    for (int j = 0; j < NR; ++j) h[t][j][0] = bias1[t];
  for (int g0 = 0; g0 < KG1; g0 += KC) {
    const int kn = KG1 - g0 < KC ? KG1 - g0 : KC;
    if (g0 != 0) __syncthreads();   // every wave is done with the previous features
    for (int g = wave; g < kn; g += 4)
#pragma unroll
      for (int j = 0; j < NR; ++j) hs[(g * NR + j) * 64 + lane] = feats16(a, c[j], g0 + g, q);
    __syncthreads();
    layer16_lds<TQ, NR, 1, 2>((const f32x4*)a.W[0] + g0 * 64, KG1, kn, hs, T0, lane, h);
  }
  auto put = [&](f32x4 (&v)[TQ][NR][1]) {   // ReLU and exchange
    __syncthreads();   // every wave is done reading the layer's input
#pragma unroll
    for (int t = 0; t < TQ; ++t)
#pragma unroll
      for (int j = 0; j < NR; ++j) {
        f32x4 x = v[t][j][0];
#pragma unroll
        for (int r = 0; r < 4; ++r) x[r] = relu(x[r]);
        hs[((T0 + t) * NR + j) * 64 + lane] = x;
      }
    __syncthreads();
  };
  put(h);
  if constexpr (NL == 3) {
    f32x4 acc[TQ][NR][NP];
#pragma unroll
    for (int t = 0; t < TQ; ++t)
#pragma unroll
      for (int j = 0; j < NR; ++j) {
        acc[t][j][0] = *(const f32x4*)(a.bias[1] + ((T0 + t) * 4 + q) * 4);
#pragma unroll
        for (int i = 1; i < NP; ++i) acc[t][j][i] = f32x4{};
      }
    layer16_lds<TQ, NR, NP, 2>((const f32x4*)a.W[1], KGH, KGH, hs, T0, lane, acc);
#pragma unroll
    for (int t = 0; t < TQ; ++t)
#pragma unroll
      for (int j = 0; j < NR; ++j) {
        f32x4 r = acc[t][j][0];
#pragma unroll
        for (int i = 1; i < NP; ++i) r += acc[t][j][i];
        h[t][j][0] = r;
      }
    put(h);
  }
#pragma unroll
  for (int j = 0; j < NR; ++j) {
    if (wave != j) continue;   // uniform
    f32x4 acc[AT][1][NPO];
#pragma unroll
    for (int T = 0; T < AT; ++T) {
      acc[T][0][0] = *(const f32x4*)(a.bias[NL - 1] + (T * 4 + q) * 4);
#pragma unroll
      for (int i = 1; i < NPO; ++i) acc[T][0][i] = f32x4{};
    }
    layer16_out<AT, NR, NPO, 4>((const f32x4*)a.W[NL - 1], KGH, hs + j * 64, lane, acc);
    f32x4 out[AT];
#pragma unroll
    for (int T = 0; T < AT; ++T) {
      out[T] = acc[T][0][0];
      if constexpr (NPO == 4) out[T] = (out[T] + acc[T][0][1]) + (acc[T][0][2] + acc[T][0][3]);
    }
    epilogue16<AT>(c[j], out, q);
  }
}
// The blocks that n rows take on a device of `cus` compute units (0: not known):
// `pairs` of two 16-row tiles, then `singles` of one.
//
// One tile per block while the blocks fit one per compute unit (a block's latency
// bounds the launch), else two, which halves the weight bytes from L2 per MFMA. us
// per launch at 1 / 2 tiles: 86 -> 256 -> 256 -> 15 at 4,096 rows 12.5 / 17.8,
// 8,192 rows 21.2 / 18.4, 16,384 rows 37.8 / 32.7; 449 -> 256 -> 64 at 4,096 rows
// 22.6 / 30.8, 16,384 rows 58.0 / 49.4.
// With two, the rows past the last whole round of 32-row blocks (one per compute
// unit) go in 16-row blocks if these fit one per compute unit: a few rows more than
// whole rounds then cost their units half a block. us per launch with 32-row blocks
// only / with the tail in 16-row blocks, 86 -> 256 -> 256 -> 15: 8,250 rows 30.9 /
// 26.2, 16,400 rows 43.0 / 37.5, 20,480 rows 45.6 / 40.4, 33,000 rows 74.7 / 66.1;
// 54 -> 64 -> 15: 16,400 rows 7.2 / 6.7. Past half a round the tail would need two
// 16-row blocks on some units, which a 32-row block does in less time.
struct F32Blocks {
  int32_t pairs, singles;
};
__host__ __device__ inline F32Blocks f32_blocks(int32_t n, int32_t cus) {
  if (cus <= 0 || n <= 16 * cus) return {0, (n + 15) / 16};
  const int32_t rest = n % (32 * cus);
  if (rest > 16 * cus) return {(n + 31) / 32, 0};
  return {(n - rest) / 32, (rest + 15) / 16};
}

// NR 2: the first a.pair_blocks blocks take 32 rows, the others 16. Chain pools:
// the row count is known here only, and the blocks are shared out by it (the
// launch's grid covers every count up to the bound).
template <int H, int NL, int AT, int NR>
__global__ __launch_bounds__(256) void route_f32s(RouteArgs a_in) {
  // chain pools: the tick's row count is on the device
  RouteArgs a = a_in;
  if (a_in.n_total_dev) a.n_total = min(*a_in.n_total_dev, a_in.n_total);   // the caller's buffers bound it
  __shared__ f32x4 hs[kF32Groups<H> * NR * 64];
  const int32_t b = (int32_t)blockIdx.x;
  if constexpr (NR == 1) {
    f32s_block<H, NL, AT, 1>(a, 16 * b, hs);
  } else {
    const int32_t pairs = a_in.n_total_dev ? f32_blocks(a.n_total, a.cus).pairs : a.pair_blocks;
    if (b < pairs) {   // uniform
      f32s_block<H, NL, AT, 2>(a, 32 * b, hs);
    } else {
      f32s_block<H, NL, AT, 1>(a, 16 * (pairs + b), hs);
    }
  }
}

// ---------------------------------------------------------------------------
// Persistent variant for policies whose deeper layers fit in LDS.
//
// Each block (NW waves) copies the packed weights of layers >= 2 (and of
// layer 1 when it also fits) into LDS once, then its waves take turns over
// the block's share of wave tiles. A wave tile is NR 32-row MFMA column tiles,
// so every weight fragment read feeds NR MFMAs. Layer-1 outputs are produced
// one 32-feature tile at a time and rounded to bf16 fragments right away.
// ---------------------------------------------------------------------------

// Copies n 16-byte words from global memory to LDS with `nthreads` threads,
// batches of 8 loads in flight per thread.
template <int N, int NTHREADS>
__device__ __forceinline__ void copy_to_lds(u32x4* dst, const u32x4* src) {
  constexpr int PER = (N + NTHREADS - 1) / NTHREADS;
  constexpr int B = 8;
#pragma unroll
  for (int b0 = 0; b0 < PER; b0 += B) {
    u32x4 v[B];
#pragma unroll
    for (int j = 0; j < B; ++j) {
      const int i = (b0 + j) * NTHREADS + (int)threadIdx.x;
      if (b0 + j < PER && i < N) v[j] = src[i];
    }
#pragma unroll
    for (int j = 0; j < B; ++j) {
      const int i = (b0 + j) * NTHREADS + (int)threadIdx.x;
      if (b0 + j < PER && i < N) dst[i] = v[j];
    }
  }
}

// Wave tiles (32 NR rows each) of block b in a persistent grid of G blocks:
// the contiguous range [first, end) of an equal split of all n_units (the
// shares differ by at most one tile). A row count just above a multiple of
// the grid's capacity then adds one tile to a few blocks instead of a whole
// extra round of tiles to one block.
struct UnitRange {
  int32_t first, end;
};
__device__ __forceinline__ UnitRange block_units(int32_t n_units) {
  UnitRange u;
  u.first = (int32_t)(((int64_t)blockIdx.x * n_units) / gridDim.x);
  u.end = (int32_t)(((int64_t)(blockIdx.x + 1) * n_units) / gridDim.x);
  return u;
}

template <int H, int NL, int AT, int KB1, bool W1L, int NW, int ED, int NR, int RL, int W1PF, bool PIPE>
__global__ __launch_bounds__(NW * 64, 1) void route_bf16_lds(RouteArgs a_in) {
  // chain pools: the tick's row count is on the device
  RouteArgs a = a_in;
  if (a_in.n_total_dev) a.n_total = min(*a_in.n_total_dev, a_in.n_total);   // the caller's buffers bound it
  constexpr int TH = H / 32;
  constexpr int KH = H / 16;
  constexpr int N_W1 = TH * KB1 * 64;
  constexpr int N_W2 = (NL == 3 ? TH : AT) * KH * 64;
  constexpr int N_W3 = NL == 3 ? AT * KH * 64 : 0;
  constexpr int N_LDS = (W1L ? N_W1 : 0) + N_W2 + N_W3;
  // biases in accumulator-register order: [tile][g][16] floats per layer
  constexpr int NB0 = TH * 32, NB1 = (NL == 3 ? TH : AT) * 32, NB2 = NL == 3 ? AT * 32 : 0;
  constexpr int WROWS = 32 * NR;            // rows per wave tile
  __shared__ u32x4 lds[N_LDS];
  __shared__ float lbias[NB0 + NB1 + NB2];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // wave-uniform loop control
  const int n = lane & 31, g = lane >> 5;
  const UnitRange ur = block_units((a.n_total + WROWS - 1) / WROWS);
  // Wave tile u is set up in two steps: its first loads (the CSR window and
  // the rows' q_idx and budget), then, once they have arrived, the env
  // lookup, the env's snapshot row and the embedding rows (row contexts and
  // layer-1 B fragments). A 64-row tile has a row per lane: each lane looks its
  // own row up and hands the two MFMA tiles what their gathers need.
  constexpr int NC = NR == 2 ? 1 : NR;      // row contexts per lane
  struct First {
    EnvWindow w;
    int32_t q[NC], bud[NC];
  };
  auto first_loads = [&](int32_t u) {
    First f;
    const int32_t r0 = u * WROWS;
    f.w = env_window(a, r0);
#pragma unroll
    for (int j = 0; j < NC; ++j) {
      const int32_t r = r0 + 32 * j + (NR == 2 ? lane : n);
      const int32_t rr = r < a.n_total ? r : a.n_total - 1;
      f.q[j] = a.q_idx[rr];
      f.bud[j] = a.budget[rr];
    }
    return f;
  };
  auto setup = [&](int32_t u, const First& f, RowCtx (&c)[NC], u32x4 (&x)[NR][KB1], int gg) {
    const int32_t r0 = u * WROWS;
    const int32_t rlast = (r0 + WROWS - 1 < a.n_total ? r0 + WROWS - 1 : a.n_total - 1);
    int32_t rows[NC], envs[NC];
#pragma unroll
    for (int j = 0; j < NC; ++j) rows[j] = r0 + 32 * j + (NR == 2 ? lane : n);
    find_envs_in<NC>(a, f.w, r0, rlast, rows, envs);
#pragma unroll
    for (int j = 0; j < NC; ++j) c[j] = row_ctx_from(a, rows[j], envs[j], f.q[j], f.bud[j]);
    TailRaw<ED, KB1> raw[NR];
    RowCtx t[NR];   // what the gathers read
    if constexpr (NR == 2) {
      int32_t tq[2], te[2], tb[2];
      spread(c[0].q, tq);
      spread(c[0].e, te);
      spread(c[0].budget, tb);
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        t[j].q = tq[j];
        t[j].e = te[j];
        t[j].budget = tb[j];
      }
    } else {
#pragma unroll
      for (int j = 0; j < NR; ++j) t[j] = c[j];
    }
#pragma unroll
    for (int j = 0; j < NR; ++j) gather_issue<ED, KB1>(a, t[j], gg, x[j], raw[j]);
#pragma unroll
    for (int j = 0; j < NR; ++j) gather_finish<ED, KB1>(a, t[j], gg, x[j], raw[j]);
  };
  // PIPE: the first wave tile is set up (first loads, then its gather)
  // while the block copies the weights into LDS, before the barrier, and each
  // later tile at the end of the previous iteration, so the loop starts with
  // layer 1 (its inputs are loop-carried: this pays only where the registers
  // are not all taken).
  int32_t u = ur.first + wave;
  RowCtx c[NC];
  u32x4 x[NR][KB1];
  First f0;
  if (PIPE && u < ur.end) f0 = first_loads(u);
  if constexpr (W1L) copy_to_lds<N_W1, NW * 64>(lds, (const u32x4*)a.W[0]);
  copy_to_lds<N_W2, NW * 64>(lds + (W1L ? N_W1 : 0), (const u32x4*)a.W[1]);
  if constexpr (NL == 3) copy_to_lds<N_W3, NW * 64>(lds + (W1L ? N_W1 : 0) + N_W2, (const u32x4*)a.W[2]);
  for (int i = threadIdx.x; i < NB0 + NB1 + NB2; i += NW * 64)
    lbias[i] = i < NB0 ? a.bias[0][i] : (i < NB0 + NB1 ? a.bias[1][i - NB0] : a.bias[2][i - NB0 - NB1]);
  if constexpr (PIPE) {
    if (u < ur.end) setup(u, f0, c, x, g);
  }
  __syncthreads();
  if (u >= ur.end) return;
  const float* lb0 = lbias;
  const float* lb1 = lbias + NB0;
  const float* lb2 = lbias + NB0 + NB1;
  const u32x4* w1 = W1L ? (const u32x4*)lds : (const u32x4*)a.W[0];
  const u32x4* w2 = lds + (W1L ? N_W1 : 0);
  const u32x4* w3 = w2 + N_W2;

  for (;;) {
    // Keeps loop-invariant loads (biases, weights) inside the loop: hoisted
    // out of it they would stay live in registers for the whole kernel.
    asm volatile("" ::: "memory");
    // Per-iteration copies of the lane index: every fragment address derived
    // from them is recomputed inside the iteration instead of being hoisted
    // (and kept live) across the whole loop.
    int ln = lane, gg = g;
    asm volatile("" : "+v"(ln), "+v"(gg));
    if constexpr (!PIPE) setup(u, first_loads(u), c, x, gg);

    u32x4 h[NR][NL == 3 ? KH : 1];
    // two-layer policies: the output layer consumes each layer-1 output tile
    // as soon as it is rounded (its two K steps), so the hidden layer is
    // never held whole
    f32x16 o[NR][AT];
    if constexpr (NL == 2) {
#pragma unroll
      for (int T = 0; T < AT; ++T) {
        o[0][T] = *(const f32x16*)(lb1 + (T * 2 + gg) * 16);
#pragma unroll
        for (int j = 1; j < NR; ++j) o[j][T] = o[0][T];
      }
    }
    // layer-1 fragments: W1PF of the next output tile's K steps are loaded
    // while the current tile's MFMAs run (the rest just before they are used)
    u32x4 wk[KB1], wn[KB1];
#pragma unroll
    for (int kb = 0; kb < KB1; ++kb) wn[kb] = w1[kb * 64 + ln];
#pragma unroll
    for (int cc = 0; cc < TH; ++cc) {
#pragma unroll
      for (int kb = 0; kb < KB1; ++kb) wk[kb] = kb < W1PF || cc == 0 ? wn[kb] : w1[(cc * KB1 + kb) * 64 + ln];
      if (cc + 1 < TH) {
#pragma unroll
        for (int kb = 0; kb < W1PF; ++kb) wn[kb] = w1[((cc + 1) * KB1 + kb) * 64 + ln];
      }
      f32x16 p[NR];
      p[0] = *(const f32x16*)(lb0 + (cc * 2 + gg) * 16);
#pragma unroll
      for (int j = 1; j < NR; ++j) p[j] = p[0];
#pragma unroll
      for (int kb = 0; kb < KB1; ++kb) {
#pragma unroll
        for (int j = 0; j < NR; ++j) p[j] = mfma_bf16(wk[kb], x[j][kb], p[j]);
      }
      if constexpr (NL == 2) {
        u32x4 f[NR][2];
#pragma unroll
        for (int j = 0; j < NR; ++j) relu_to_frags(p[j], f[j][0], f[j][1]);
#pragma unroll
        for (int T = 0; T < AT; ++T) {
          const u32x4 wa = w2[(T * KH + 2 * cc) * 64 + ln];
          const u32x4 wb = w2[(T * KH + 2 * cc + 1) * 64 + ln];
#pragma unroll
          for (int j = 0; j < NR; ++j) {
            o[j][T] = mfma_bf16(wa, f[j][0], o[j][T]);
            o[j][T] = mfma_bf16(wb, f[j][1], o[j][T]);
          }
        }
      } else {
#pragma unroll
        for (int j = 0; j < NR; ++j) relu_to_frags(p[j], h[j][2 * cc], h[j][2 * cc + 1]);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (NL == 3) {
#pragma unroll
      for (int T = 0; T < AT; ++T) {
        o[0][T] = *(const f32x16*)(lb2 + (T * 2 + gg) * 16);
#pragma unroll
        for (int j = 1; j < NR; ++j) o[j][T] = o[0][T];
      }
#pragma unroll
      for (int cc = 0; cc < TH; ++cc) {
        f32x16 p[NR];
        p[0] = *(const f32x16*)(lb1 + (cc * 2 + gg) * 16);
#pragma unroll
        for (int j = 1; j < NR; ++j) p[j] = p[0];
        // LDS fragments two K steps ahead of the MFMAs that use them
        u32x4 w_0 = w2[(cc * KH + 0) * 64 + ln];
        u32x4 w_1 = w2[(cc * KH + 1) * 64 + ln];
        // the wave raises its issue priority for the chain of MFMAs, so that
        // the other wave of its SIMD runs its ReLU, packing and loads in the
        // chain's shadow instead of taking turns on the matrix pipe
        if constexpr (!PIPE && NR == 2) __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int kb = 0; kb < KH; ++kb) {
          const u32x4 w_2 = w2[(cc * KH + (kb + 2 < KH ? kb + 2 : KH - 1)) * 64 + ln];
#pragma unroll
          for (int j = 0; j < NR; ++j) p[j] = mfma_bf16(w_0, h[j][kb], p[j]);
          w_0 = w_1;
          w_1 = w_2;
          __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (!PIPE && NR == 2) __builtin_amdgcn_s_setprio(0);
        u32x4 f[NR][2];
#pragma unroll
        for (int j = 0; j < NR; ++j) relu_to_frags(p[j], f[j][0], f[j][1]);
#pragma unroll
        for (int To = 0; To < AT; ++To) {
          const u32x4 wa = w3[(To * KH + 2 * cc) * 64 + ln];
          const u32x4 wb = w3[(To * KH + 2 * cc + 1) * 64 + ln];
#pragma unroll
          for (int j = 0; j < NR; ++j) {
            o[j][To] = mfma_bf16(wa, f[j][0], o[j][To]);
            o[j][To] = mfma_bf16(wb, f[j][1], o[j][To]);
          }
        }
      }
    }
    const int32_t un = u + NW;
    if constexpr (NR == 2) {
      epilogue64<AT, RL>(c[0], o, gg);
    } else {
#pragma unroll
      for (int j = 0; j < NR; ++j) epilogue<AT, RL>(c[j], o[j], gg);
    }
    if (un >= ur.end) break;
    u = un;
    if constexpr (PIPE) setup(u, first_loads(u), c, x, gg);
  }
}

// ---------------------------------------------------------------------------
// Streaming variant for wide three-layer policies whose weights do not fit in
// LDS (c3: 193 -> 512 -> 512 -> 64, 784 KB in bf16).
//
// A block of NW waves routes NW x 32 rows per step; each wave keeps its
// rows' whole first hidden layer in registers as bf16 B fragments. The
// weights pass through a double-buffered LDS ring in stages: two layer-1
// output tiles, or one layer-2 output tile together with the layer-3
// fragments that consume it (layer-2 outputs are never stored). The next
// stage is brought in by the LDS DMA path (global_load_lds, no registers)
// while the current one is multiplied; one barrier per stage.
// ---------------------------------------------------------------------------

// 16 floats from LDS as four 16-byte reads (each keeps the LDS variable's
// alias information, which a single 64-byte access loses when it is split).
__device__ __forceinline__ f32x16 lds_f32x16(const u32x4* p) {
  const u32x4 v0 = p[0], v1 = p[1], v2 = p[2], v3 = p[3];
  f32x16 r;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    r[i] = __uint_as_float(v0[i]);
    r[4 + i] = __uint_as_float(v1[i]);
    r[8 + i] = __uint_as_float(v2[i]);
    r[12 + i] = __uint_as_float(v3[i]);
  }
  return r;
}

template <int H, int AT, int KB1, int ED, int NW, int RL>
__global__ __launch_bounds__(NW * 64, 1) void route_bf16_stream(RouteArgs a_in) {
  // chain pools: the tick's row count is on the device
  RouteArgs a = a_in;
  if (a_in.n_total_dev) a.n_total = min(*a_in.n_total_dev, a_in.n_total);   // the caller's buffers bound it
  constexpr int TH = H / 32, KH = H / 16;
  constexpr int S1 = TH / 2;                  // layer-1 stages (two output tiles each)
  constexpr int NST = S1 + TH;                // stages per block step
  constexpr int F1 = 2 * KB1;                 // fragments of a layer-1 stage
  constexpr int F2 = KH + 2 * AT;             // fragments of a layer-2 stage
  constexpr int FS = F1 > F2 ? F1 : F2;
  constexpr int NB0 = TH * 32, NB1 = TH * 32, NB2 = AT * 32;
  static_assert(NST % 2 == 0, "stage parity must repeat every block step");
  static_assert(KH % NW == 0 && 2 * AT <= NW, "layer-2 stage split over the waves");
  // Two separately declared buffers, each with its own copy of the biases
  // behind the weight fragments: a stage reads only the buffer the copy in
  // flight does not target, which the compiler can then tell apart (with one
  // array it waits for the next stage's copy before every read).
  constexpr int NBW = (NB0 + NB1 + NB2) / 4;   // biases in 16-byte words
  static_assert((NB0 + NB1 + NB2) % 4 == 0, "bias rows move in 16-byte words");
  __shared__ u32x4 ring0[FS * 64 + NBW];
  __shared__ u32x4 ring1[FS * 64 + NBW];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int g = lane >> 5;
  const u32x4* W1 = (const u32x4*)a.W[0];
  const u32x4* W2 = (const u32x4*)a.W[1];
  const u32x4* W3 = (const u32x4*)a.W[2];
  // Fragments of stage st into ring buffer b: wave wv copies fragments
  // wv, wv + NW, ...; a wave with fewer fragments than the others copies the
  // stage's last one again (the same bytes to the same place), so the code
  // has no branches.
  auto issue = [&](int st, int b, int wv, int ln) {
    u32x4* dst = b ? ring1 : ring0;
    if (st < S1) {
#pragma unroll
      for (int i = 0; i < (F1 + NW - 1) / NW; ++i) {
        const int f = min(wv + NW * i, F1 - 1);
        dma_frag(dst + f * 64, W1 + (st * F1 + f) * 64, ln);
      }
    } else {
      const int j = st - S1;
#pragma unroll
      for (int i = 0; i < KH / NW; ++i) {
        const int f = wv + NW * i;
        dma_frag(dst + f * 64, W2 + (j * KH + f) * 64, ln);
      }
      const int f3 = min(wv, 2 * AT - 1);   // layer-3 fragment (To, 2 j + d) with f3 = 2 To + d
      dma_frag(dst + (KH + f3) * 64, W3 + ((f3 >> 1) * KH + 2 * j + (f3 & 1)) * 64, ln);
    }
  };
  for (int i = threadIdx.x; i < NB0 + NB1 + NB2; i += NW * 64) {
    const float v = i < NB0 ? a.bias[0][i] : (i < NB0 + NB1 ? a.bias[1][i - NB0] : a.bias[2][i - NB0 - NB1]);
    ((float*)(ring0 + FS * 64))[i] = v;
    ((float*)(ring1 + FS * 64))[i] = v;
  }
  issue(0, 0, __builtin_amdgcn_readfirstlane(wave), lane);
  // The block takes an equal contiguous share of the 32-row wave tiles (the
  // shares differ by at most one), NW per block step; in its last step the
  // waves without a tile still bring in their share of the weights and join
  // the barriers, but skip the arithmetic.
  const UnitRange ur = block_units((a.n_total + 31) / 32);
  const int n_steps = (ur.end - ur.first + NW - 1) / NW;
  for (int step = 0; step < n_steps; ++step) {
    // Per-iteration copies of the lane and wave indices: the fragment and
    // bias addresses derived from them are recomputed in each block step
    // instead of being hoisted out of the loop and kept live across it.
    asm volatile("" ::: "memory");
    int ln = lane, gg = g;
    int wv = __builtin_amdgcn_readfirstlane(wave);
    asm volatile("" : "+v"(ln), "+v"(gg));
    asm volatile("" : "+s"(wv));
    const int32_t unit = ur.first + step * NW + wv;
    const bool act = unit < ur.end;                             // wave-uniform
    const int32_t r0 = act ? unit * 32 : a.n_total - 1;        // idle waves: a clamped row, nothing stored
    const int32_t rl = r0 + 31 < a.n_total ? r0 + 31 : a.n_total - 1;
    const int32_t rows[1] = {act ? r0 + (ln & 31) : a.n_total};
    const int32_t rsel[1] = {rows[0] < a.n_total ? rows[0] : a.n_total - 1};
    int32_t envs[1];
    RowCtx c;
    u32x4 x[KB1];
    if (act) {
      find_envs<1>(a, r0, rl, rsel, envs);
      c = row_setup_env(a, rows[0], envs[0]);
      TailRaw<ED, KB1> raw;
      gather_issue<ED, KB1>(a, c, gg, x, raw);
      gather_finish<ED, KB1>(a, c, gg, x, raw);
    }
    if (!act) {
      // the same stages, barriers and copies as a working wave (a barrier
      // counts waves, wherever they wait), without the arithmetic
      for (int s = 0; s < NST; ++s) {
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        int lns = ln;
        asm volatile("" : "+v"(lns));
        issue(s + 1 < NST ? s + 1 : 0, (s + 1) & 1, wv, lns);
      }
      continue;
    }
    u32x4 h[KH];
    f32x16 z[AT];
#pragma unroll
    for (int s = 0; s < NST; ++s) {
      // stage s is in buffer s & 1; every wave is done with buffer (s + 1) & 1
      __builtin_amdgcn_s_waitcnt(0);
      __syncthreads();
      {
        // the DMA source addresses are formed here, not hoisted to the step's start
        int lns = ln;
        asm volatile("" : "+v"(lns));
        issue(s + 1 < NST ? s + 1 : 0, (s + 1) & 1, wv, lns);
      }
      const u32x4* wb = (s & 1) ? ring1 : ring0;
      const u32x4* lb4 = wb + FS * 64;   // biases, 4 floats per word
      if (s < S1) {
        // fragment q = t * KB1 + kb, two LDS reads ahead of its MFMA
        u32x4 w_0 = wb[0 * 64 + ln];
        u32x4 w_1 = wb[1 * 64 + ln];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          const int T = 2 * s + t;
          f32x16 p = lds_f32x16(lb4 + (T * 2 + gg) * 4);
#pragma unroll
          for (int kb = 0; kb < KB1; ++kb) {
            const int q = t * KB1 + kb;
            const u32x4 w_2 = wb[(q + 2 < F1 ? q + 2 : F1 - 1) * 64 + ln];
            p = mfma_bf16(w_0, x[kb], p);
            w_0 = w_1;
            w_1 = w_2;
            __builtin_amdgcn_sched_barrier(0);
          }
          relu_to_frags(p, h[2 * T], h[2 * T + 1]);
        }
        if (s == S1 - 1) {
#pragma unroll
          for (int To = 0; To < AT; ++To) z[To] = lds_f32x16(lb4 + (NB0 + NB1) / 4 + (To * 2 + gg) * 4);
        }
      } else {
        const int j = s - S1;
        f32x16 p = lds_f32x16(lb4 + NB0 / 4 + (j * 2 + gg) * 4);
        u32x4 w_0 = wb[0 * 64 + ln];
        u32x4 w_1 = wb[1 * 64 + ln];
#pragma unroll
        for (int kb = 0; kb < KH; ++kb) {
          const u32x4 w_2 = wb[(kb + 2 < F2 ? kb + 2 : F2 - 1) * 64 + ln];
          p = mfma_bf16(w_0, h[kb], p);
          w_0 = w_1;
          w_1 = w_2;
          __builtin_amdgcn_sched_barrier(0);
        }
        u32x4 f0, f1;
        relu_to_frags(p, f0, f1);
        // w_0, w_1 now hold fragments KH and KH + 1 (layer 3, To = 0)
#pragma unroll
        for (int To = 0; To < AT; ++To) {
          const u32x4 wa = To == 0 ? w_0 : wb[(KH + 2 * To) * 64 + ln];
          const u32x4 wc = To == 0 ? w_1 : wb[(KH + 2 * To + 1) * 64 + ln];
          z[To] = mfma_bf16(wa, f0, z[To]);
          z[To] = mfma_bf16(wc, f1, z[To]);
        }
      }
    }
    epilogue<AT, RL>(c, z, gg);
  }
  __builtin_amdgcn_s_waitcnt(0);   // the prefetched first stage of a step that does not exist
}

// ---------------------------------------------------------------------------
// The paper's dual-pathway executor (Sec. 4.2), persistent, on MFMA.
//
// Per request: a semantic pathway LN(ReLU(W_sem [e_q | e_r])) (128), a
// resource pathway LN(ReLU(W_res [h_bud | h_sys])) (64) over a budget head and
// a system head (16 each), a merge layer ReLU(W_merge [h_sem | h_res]) (128)
// and the action/value rows. The role half of the semantic layer takes only
// n_roles distinct inputs, so its products (plus b_sem) are computed once per
// pool (role_projection_kernel) and enter as the accumulator's initial value;
// the per-request semantic work is the 128 x E_d query half.
//
// A wave owns NR x 32 rows. The query-half, merge and action weights live in
// LDS (152 KB at E_d = 384); the small resource-layer fragments, the system
// head and the role projections are read through the caches. The query half
// of W_sem is packed so that each lane reads its row's embedding in 64-byte
// runs: within a 64-element group, lane half g takes elements 32 g .. 32 g + 31
// as four K steps of 8, so the two lanes of a row consume one 128-byte line
// per group. Groups are prefetched one ahead of the MFMAs that use them.
// ---------------------------------------------------------------------------

// fp32 -> bf16 (round to nearest even) -> fp32.
__device__ __forceinline__ float bf16_round(float x) { return __uint_as_float(pack2(x, 0.f) << 16); }

// ReLU, then LayerNorm over the 32 NT features a lane pair (n, n + 32) holds
// in NT accumulator tiles: (u - mean) / sqrt(var + 1e-5) * gain + bias with
// the biased variance, rounded to bf16 B fragments for the next layer
// (fragment 2T + h holds registers 8h .. 8h + 7 of tile T).
template <int NT>
__device__ __forceinline__ void relu_ln_frags(f32x16 (&acc)[NT], const float* gain, const float* bias,
                                              int g, u32x4 (&f)[2 * NT]) {
  constexpr float inv_n = 1.f / (32 * NT);
  float s = 0.f;
#pragma unroll
  for (int T = 0; T < NT; ++T) {
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      acc[T][v] = relu(acc[T][v]);
      s += acc[T][v];
    }
  }
  s += __shfl_xor(s, 32, 64);
  const float mean = s * inv_n;
  float q = 0.f;
#pragma unroll
  for (int T = 0; T < NT; ++T) {
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const float d = acc[T][v] - mean;
      q = fmaf(d, d, q);
    }
  }
  q += __shfl_xor(q, 32, 64);
  const float rstd = rsqrtf(fmaf(q, inv_n, 1e-5f));
#pragma unroll
  for (int T = 0; T < NT; ++T) {
    // one tile's gains and biases at a time: loads hoisted above this point
    // would keep all of them live at once
    asm volatile("" ::: "memory");
    float y[16];
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int i = (T * 2 + g) * 16 + v;
      y[v] = fmaf((acc[T][v] - mean) * rstd, gain[i], bias[i]);
    }
    f[2 * T].x = pack2(y[0], y[1]);     f[2 * T].y = pack2(y[2], y[3]);
    f[2 * T].z = pack2(y[4], y[5]);     f[2 * T].w = pack2(y[6], y[7]);
    f[2 * T + 1].x = pack2(y[8], y[9]);   f[2 * T + 1].y = pack2(y[10], y[11]);
    f[2 * T + 1].z = pack2(y[12], y[13]); f[2 * T + 1].w = pack2(y[14], y[15]);
    // the tile's fragments are complete before the next tile's loads issue
    asm volatile("" : "+v"(f[2 * T]), "+v"(f[2 * T + 1]));
  }
}

// The 4 K-step fragments of 64-element group G of a row's query embedding.
template <int ED>
__device__ __forceinline__ void load_group(const RouteArgs& a, const RowCtx& c, int G, int g, u32x4 (&x)[4]) {
  const u32x4* src = (const u32x4*)((const uint16_t*)a.emb + (size_t)c.q * ED + 64 * G + 32 * g);
#pragma unroll
  for (int i = 0; i < 4; ++i) x[i] = src[i];
}

// 64-element embedding groups in flight ahead of the MFMAs
constexpr int kDualPrefetch = 1;

template <int ED, int NW, int NR, int RL>
__global__ __launch_bounds__(NW * 64, 1) void route_dual_bf16(RouteArgs a_in) {
  // chain pools: the tick's row count is on the device
  RouteArgs a = a_in;
  if (a_in.n_total_dev) a.n_total = min(*a_in.n_total_dev, a_in.n_total);   // the caller's buffers bound it
  static_assert(ED % 64 == 0, "embedding width must be a multiple of 64");
  constexpr int KBQ = ED / 16;          // K steps of the query half
  constexpr int NG = ED / 64;           // 64-element groups
  constexpr int N_SEM = 4 * KBQ * 64;   // 16-byte fragments
  constexpr int N_MRG = 4 * 12 * 64;
  constexpr int N_ACT = 8 * 64;
  constexpr int WROWS = 32 * NR;
  __shared__ u32x4 lds[N_SEM + N_MRG + N_ACT];
  __shared__ float lp[DP_LDS];
  copy_to_lds<N_SEM, NW * 64>(lds, (const u32x4*)a.W[0]);
  copy_to_lds<N_MRG, NW * 64>(lds + N_SEM, (const u32x4*)a.W[1]);
  copy_to_lds<N_ACT, NW * 64>(lds + N_SEM + N_MRG, (const u32x4*)a.W[2]);
  for (int i = threadIdx.x; i < DP_LDS; i += NW * 64) lp[i] = a.dual_p[i];
  __syncthreads();
  const u32x4* wsem = lds;
  const u32x4* wmrg = lds + N_SEM;
  const u32x4* wact = wmrg + N_MRG;
  const u32x4* wres = (const u32x4*)a.W_res;
  const float* proj = a.dual_p + DP_ROLE;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int n = lane & 31, g = lane >> 5;
  const int n3 = 3 * a.M;
  const int sstride = snap_stride(a.M);
  const UnitRange ur = block_units((a.n_total + WROWS - 1) / WROWS);

  for (int32_t u = ur.first + wave; u < ur.end; u += NW) {
    asm volatile("" ::: "memory");
    int ln = lane, gg = g;
    asm volatile("" : "+v"(ln), "+v"(gg));
    const int32_t r0 = u * WROWS;
    const int32_t rlast = (r0 + WROWS - 1 < a.n_total ? r0 + WROWS - 1 : a.n_total - 1);
    int32_t rows[NR], envs[NR];
#pragma unroll
    for (int j = 0; j < NR; ++j) rows[j] = r0 + 32 * j + n;
    find_envs<NR>(a, r0, rlast, rows, envs);
    RowCtx c[NR];
    int32_t role[NR];
#pragma unroll
    for (int j = 0; j < NR; ++j) {
      c[j] = row_setup_env(a, rows[j], envs[j]);
      const int32_t ro = a.role[c[j].live ? rows[j] : a.n_total - 1];
      const bool bad_r = ro < 0 || ro >= a.n_roles;
      if (bad_r) c[j].bad |= IM_ERR_ROLE;
      role[j] = bad_r ? 0 : ro;
    }

    // ---- semantic pathway: role projection + W_sem (query half) e_q ----
    // ring of PF + 1 groups: group G + PF is loaded while group G is multiplied
    constexpr int PF = kDualPrefetch < NG ? kDualPrefetch : NG - 1;
    u32x4 x[PF + 1][NR][4];
#pragma unroll
    for (int G = 0; G < PF; ++G) {
#pragma unroll
      for (int j = 0; j < NR; ++j) load_group<ED>(a, c[j], G, gg, x[G][j]);
    }
    // ---- resource pathway, computed while the first embedding groups load ----
    u32x4 hr[NR][4];
#pragma unroll
    for (int j = 0; j < NR; ++j) {
      // budget head: features 8 gg .. 8 gg + 7 of h_bud (K step 0 of W_res)
      const float bfe = bf16_round((float)c[j].budget * a.inv_bud);
      float hb[8], hy[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        hb[k] = relu(fmaf(lp[DP_W_BUD + 8 * gg + k], bfe, lp[DP_B_BUD + 8 * gg + k]));
        hy[k] = lp[DP_B_SYS + 8 * gg + k];
      }
      // system head: features 8 gg .. 8 gg + 7 of h_sys (K step 1) over the
      // env's queue-depth, KV-proxy and latency features, read 8 at a time
      // (weights of the features past 3M are zero)
      const float* srow = a.snap + (size_t)c[j].e * sstride;
      for (int k0 = 0; k0 < n3; k0 += 8) {
        const float4 d0 = *(const float4*)(srow + k0);
        const float4 d1 = *(const float4*)(srow + k0 + 4);
        const float dv[8] = {d0.x, d0.y, d0.z, d0.w, d1.x, d1.y, d1.z, d1.w};
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) {
          const float d = bf16_round(dv[kk]);
          const float* w = lp + DP_W_SYS + (k0 + kk) * 16 + 8 * gg;
#pragma unroll
          for (int q = 0; q < 8; ++q) hy[q] = fmaf(w[q], d, hy[q]);
        }
      }
      u32x4 f0, f1;
      f0.x = relu_pack2(hb[0], hb[1]); f0.y = relu_pack2(hb[2], hb[3]);
      f0.z = relu_pack2(hb[4], hb[5]); f0.w = relu_pack2(hb[6], hb[7]);
      f1.x = relu_pack2(hy[0], hy[1]); f1.y = relu_pack2(hy[2], hy[3]);
      f1.z = relu_pack2(hy[4], hy[5]); f1.w = relu_pack2(hy[6], hy[7]);
      f32x16 rr[2];
#pragma unroll
      for (int T = 0; T < 2; ++T) {
        rr[T] = *(const f32x16*)(lp + DP_B_RES + (T * 2 + gg) * 16);
        rr[T] = mfma_bf16(wres[(T * 2 + 0) * 64 + ln], f0, rr[T]);
        rr[T] = mfma_bf16(wres[(T * 2 + 1) * 64 + ln], f1, rr[T]);
      }
      relu_ln_frags<2>(rr, lp + DP_LN_RES_G, lp + DP_LN_RES_B, gg, hr[j]);
    }
    __builtin_amdgcn_sched_barrier(0);

    f32x16 s[NR][4];
#pragma unroll
    for (int j = 0; j < NR; ++j) {
#pragma unroll
      for (int T = 0; T < 4; ++T) s[j][T] = *(const f32x16*)(proj + ((role[j] * 4 + T) * 2 + gg) * 16);
    }
#pragma unroll
    for (int G = 0; G < NG; ++G) {
      if (G + PF < NG) {
#pragma unroll
        for (int j = 0; j < NR; ++j) load_group<ED>(a, c[j], G + PF, gg, x[(G + PF) % (PF + 1)][j]);
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int kb = 4 * G + i;
#pragma unroll
        for (int T = 0; T < 4; ++T) {
          const u32x4 w = wsem[(T * KBQ + kb) * 64 + ln];
#pragma unroll
          for (int j = 0; j < NR; ++j) s[j][T] = mfma_bf16(w, x[G % (PF + 1)][j][i], s[j][T]);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    u32x4 hs[NR][8];
#pragma unroll
    for (int j = 0; j < NR; ++j) relu_ln_frags<4>(s[j], lp + DP_LN_SEM_G, lp + DP_LN_SEM_B, gg, hs[j]);
    __builtin_amdgcn_sched_barrier(0);

    // ---- decision: merge layer, then the action/value rows ----
    u32x4 hh[NR][8];
#pragma unroll
    for (int T = 0; T < 4; ++T) {
      f32x16 m[NR];
      m[0] = *(const f32x16*)(lp + DP_B_MERGE + (T * 2 + gg) * 16);
#pragma unroll
      for (int j = 1; j < NR; ++j) m[j] = m[0];
#pragma unroll
      for (int kb = 0; kb < 12; ++kb) {
        const u32x4 w = wmrg[(T * 12 + kb) * 64 + ln];
#pragma unroll
        for (int j = 0; j < NR; ++j) m[j] = mfma_bf16(w, kb < 8 ? hs[j][kb] : hr[j][kb - 8], m[j]);
      }
#pragma unroll
      for (int j = 0; j < NR; ++j) relu_to_frags(m[j], hh[j][2 * T], hh[j][2 * T + 1]);
      __builtin_amdgcn_sched_barrier(0);
    }
    f32x16 o[NR][1];
    o[0][0] = *(const f32x16*)(lp + DP_B_ACT + gg * 16);
#pragma unroll
    for (int j = 1; j < NR; ++j) o[j][0] = o[0][0];
#pragma unroll
    for (int kb = 0; kb < 8; ++kb) {
      const u32x4 w = wact[kb * 64 + ln];
#pragma unroll
      for (int j = 0; j < NR; ++j) o[j][0] = mfma_bf16(w, hh[j][kb], o[j][0]);
    }
#pragma unroll
    for (int j = 0; j < NR; ++j) epilogue<1, RL>(c[j], o[j], gg);
  }
}

// Role projections, one thread per (role, output feature): fp32 sum of the
// bf16 products, stored in accumulator-register order.
__global__ void role_projection_kernel(const uint16_t* w_role, const uint16_t* roles, const float* b_sem,
                                       int n_roles, int ed, float* out) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n_roles * kDualSem) return;
  const int r = i / kDualSem, o = i % kDualSem;
  float acc = b_sem[o];
  for (int k = 0; k < ed; ++k)
    acc = fmaf(bf16_to_f32(w_role[(size_t)o * ed + k]), bf16_to_f32(roles[(size_t)r * ed + k]), acc);
  // feature o = 32 T + 8 (v / 4) + 4 g + v % 4
  const int T = o >> 5, w = o & 31, v = ((w >> 3) << 2) | (w & 3), g = (w >> 2) & 1;
  out[(((size_t)r * 4 + T) * 2 + g) * 16 + v] = acc;
}

template <int H, int NL, int NR>
RouteKernel pick_f32s(int at) {
  return at == 1 ? route_f32s<H, NL, 1, NR>
                 : (at == 2 ? route_f32s<H, NL, 2, NR> : (at == 3 ? route_f32s<H, NL, 3, NR> : route_f32s<H, NL, 4, NR>));
}
template <int H, int NL>
RouteKernel pick_f32(int at, int nr) {
  // at: output tiles of 16 (fp32 pools); feature-split kernel when the hidden
  // tiles split four ways, nr row tiles per block
  if constexpr ((H / 16) % 4 == 0)
    return nr == 1 ? pick_f32s<H, NL, 1>(at) : pick_f32s<H, NL, 2>(at);
  else
    return at == 1 ? route_f32<H, NL, 1>
                   : (at == 2 ? route_f32<H, NL, 2> : (at == 3 ? route_f32<H, NL, 3> : route_f32<H, NL, 4>));
}

template <int NL>
RouteKernel pick(int hidden, int at, int nr) {
  switch (hidden) {
    case 32: return pick_f32<32, NL>(at, nr);
    case 64: return pick_f32<64, NL>(at, nr);
    case 128: return pick_f32<128, NL>(at, nr);
    case 256: return pick_f32<256, NL>(at, nr);
  }
  return nullptr;
}

// Persistent LDS-resident kernels and their launch shape (waves per block,
// 32-row MFMA tiles per wave). The greedy route and the RL outputs are
// separate instantiations, so each keeps only the registers its own epilogue
// needs.
struct LdsLaunch {
  RouteKernel k;
  int waves;   // per block
  int rows;    // 32-row MFMA tiles per wave
};

// 86 -> 256 -> 256 -> A, layer-1 weights through the caches: 8 waves (two per
// SIMD) of 64 rows, so every weight fragment read from LDS or the caches feeds
// two MFMAs and a row's setup and output run on a lane of its own, with the next
// output tile's layer-1 fragments loaded while the current one is multiplied (up
// to 256 VGPRs per wave). Light ticks, whose few tiles would leave most waves
// idle, run 16 waves of 32 rows; very light greedy ones 8 waves of 32 rows,
// software-pipelined. us, RL outputs, 32 / 64 rows per wave: 65,536 rows 17.6 /
// 19.1, 262,144 rows 50.9 / 48.1, 2,097,152 rows 368 / 319.
// 104 -> 256 -> A, every layer in LDS, software-pipelined, the output layer
// consuming each hidden tile as soon as it is produced: 12 waves (three per SIMD,
// 168 VGPRs) of 64 rows; the RL outputs below 1,024 rows per block run 16 waves
// of 32 rows. us, RL outputs, 32 / 64 rows per wave: 131,072 rows 16.8 / 17.3,
// 196,608 rows 21.4 / 22.5, 262,144 rows 27.7 / 26.2, 2,097,152 rows 180 / 172.
// Returns a null kernel when no LDS-resident variant applies.
LdsLaunch pick_lds(int dtype, int hidden, int n_layers, int out_tiles, int k1, int ed, bool rl, int light,
                   int64_t rows_per_block) {
  if (dtype != IM_BF16) return {nullptr, 0, 0};
  if (hidden == 256 && n_layers == 3 && out_tiles == 1 && k1 == 6 && ed == 64) {
    if (rl && light == 0) return {route_bf16_lds<256, 3, 1, 6, false, 8, 64, 2, 1, 6, false>, 8, 2};
    if (rl) return {route_bf16_lds<256, 3, 1, 6, false, 16, 64, 1, 1, 0, false>, 16, 1};
    if (light == 2) return {route_bf16_lds<256, 3, 1, 6, false, 8, 64, 1, 0, 6, true>, 8, 1};
    if (light == 1) return {route_bf16_lds<256, 3, 1, 6, false, 16, 64, 1, 0, 0, false>, 16, 1};
    return {route_bf16_lds<256, 3, 1, 6, false, 8, 64, 2, 0, 6, false>, 8, 2};
  }
  if (hidden == 256 && n_layers == 2 && out_tiles == 1 && k1 == 7 && ed == 64) {
    if (rl && rows_per_block < 1024) return {route_bf16_lds<256, 2, 1, 7, true, 16, 64, 1, 1, 0, true>, 16, 1};
    return {rl ? route_bf16_lds<256, 2, 1, 7, true, 12, 64, 2, 1, 0, true>
               : route_bf16_lds<256, 2, 1, 7, true, 12, 64, 2, 0, 0, true>, 12, 2};
  }
  return {nullptr, 0, 0};
}

// Streaming kernels: kStreamWaves waves per block, 32 rows per wave. The
// greedy route and the RL outputs are separate instantiations, so each keeps
// only the registers its own epilogue needs.
constexpr int kStreamWaves = 8;

RouteKernel pick_stream(int dtype, int hidden, int n_layers, int out_tiles, int k1, int ed, bool rl) {
  if (dtype != IM_BF16) return nullptr;
  if (hidden == 512 && n_layers == 3 && out_tiles == 2 && k1 == 13 && ed == 128)
    return rl ? route_bf16_stream<512, 2, 13, 128, kStreamWaves, 1>
              : route_bf16_stream<512, 2, 13, 128, kStreamWaves, 0>;
  if (hidden == 512 && n_layers == 3 && out_tiles == 3 && k1 == 13 && ed == 128)
    return rl ? route_bf16_stream<512, 3, 13, 128, kStreamWaves, 1>
              : route_bf16_stream<512, 3, 13, 128, kStreamWaves, 0>;
  return nullptr;
}

// Dual-pathway kernels: kDualWaves waves per block, kDualRows row tiles per wave.
constexpr int kDualWaves = 16;
constexpr int kDualRows = 1;

RouteKernel pick_dual(int ed, bool rl) {
  switch (ed) {
    case 64: return rl ? route_dual_bf16<64, kDualWaves, kDualRows, 1> : route_dual_bf16<64, kDualWaves, kDualRows, 0>;
    case 128: return rl ? route_dual_bf16<128, kDualWaves, kDualRows, 1> : route_dual_bf16<128, kDualWaves, kDualRows, 0>;
    case 256: return rl ? route_dual_bf16<256, kDualWaves, kDualRows, 1> : route_dual_bf16<256, kDualWaves, kDualRows, 0>;
    case 384: return rl ? route_dual_bf16<384, kDualWaves, kDualRows, 1> : route_dual_bf16<384, kDualWaves, kDualRows, 0>;
  }
  return nullptr;
}

hipError_t launch_dual(const RouteArgs& a, hipStream_t s) {
  RouteKernel k = pick_dual(a.embed_dim, a.rl != 0);
  if (!k) return hipErrorInvalidValue;
  const int rows = 32 * kDualRows;
  const int units = (a.n_total + rows - 1) / rows;   // wave tiles, spread over up to one block per CU
  const unsigned blocks =
      (unsigned)(a.persistent_blocks > 0 && units > a.persistent_blocks ? a.persistent_blocks : units);
  hipLaunchKernelGGL(k, dim3(blocks), dim3(kDualWaves * 64), 0, s, a);
  return hipGetLastError();
}

}  // namespace

bool dual_supported(int embed_dim, int out_rows) {
  return out_rows >= 1 && out_rows <= 32 && pick_dual(embed_dim, false) != nullptr;
}

hipError_t launch_role_projection(const uint16_t* w_role, const uint16_t* roles, const float* b_sem,
                                  int n_roles, int embed_dim, float* out, hipStream_t s) {
  const int n = n_roles * kDualSem;
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(role_projection_kernel, dim3((n + 255) / 256), dim3(256), 0, s, w_role, roles, b_sem,
                     n_roles, embed_dim, out);
  return hipGetLastError();
}

// out_tiles: output tiles of the last layer, 32 rows (bf16) or 16 rows (fp32).
bool route_supported(int dtype, int hidden, int n_layers, int out_tiles) {
  if (n_layers != 2 && n_layers != 3) return false;
  if (out_tiles < 1 || out_tiles > (dtype == IM_F32 ? 4 : 3)) return false;
  if (dtype == IM_BF16) return split_supported(hidden);
  return (n_layers == 2 ? pick<2>(hidden, out_tiles, 1) : pick<3>(hidden, out_tiles, 1)) != nullptr;
}

hipError_t launch_route(const RouteArgs& a, int dtype, int hidden, int n_layers, int out_tiles,
                        hipStream_t s) {
  if (a.n_total <= 0) return hipSuccess;
  if (a.net == IM_NET_DUAL) return launch_dual(a, s);
  if (!route_supported(dtype, hidden, n_layers, out_tiles)) return hipErrorInvalidValue;
  // A small tick is bound by one block's latency: the persistent kernels
  // first copy (or stream) every weight through LDS, the feature-split kernel
  // reads each fragment once and spreads a row group over all its waves. It is
  // ahead up to one 64-row block per persistent block, and for hidden width 512
  // (784 KB of weights to stream) up to one 128-row block. us, greedy,
  // persistent / split, at 8,192, 16,384, 32,768 and 65,536 rows:
  //   86 -> 256 -> 256 -> 15   9.6 / 8.0, 10.0 / 9.4, 10.9 / 12.4, 17.0 / 18.7
  //   104 -> 256 -> 24         8.7 / 6.2, 9.0 / 7.4, 9.6 / 9.2, 11.2 / 12.6
  //   193 -> 512 -> 512 -> 64  37.9 / 18.0, 38.3 / 22.3, 40.5 / 31.5, 49.1 / 59.8
  const bool persistent = pick_lds(dtype, hidden, n_layers, out_tiles, a.k1, a.embed_dim, false, 0, 0).k ||
                          pick_stream(dtype, hidden, n_layers, out_tiles, a.k1, a.embed_dim, false);   // the shape has such a kernel
  const int64_t split_rows = (int64_t)(hidden == 512 ? 128 : 64) * a.persistent_blocks;
  if (dtype == IM_BF16 && a.n_total <= split_rows) return launch_split(a, hidden, n_layers, out_tiles, !persistent, s);
  if (a.persistent_blocks > 0) {
    // a light tick (at most three 64-row tiles per four waves of 8-wave
    // blocks) runs the 16-wave, 32-row shape: twice the waves share its rows;
    // a very light one (at most one 32-row tile per two waves) runs 8 waves
    // of 32 rows whose first tile's loads overlap the block's weight copy
    // Chain pools, whose rows are not known here: greedy ticks go by the bound, RL
    // outputs by the arrivals, so that few rows under a large bound are not spread
    // over 64-row tiles (us per im_route_sample, 86 -> 256 -> 256 -> 16, by the bound
    // / by the arrivals, 22,551 rows of at most 180,224, 25.6 / 23.5).
    const int64_t rows = a.rl ? a.n_least : a.n_total, cap = (int64_t)64 * 8 * a.persistent_blocks;
    const int light = rows * 4 <= cap ? 2 : (rows * 4 <= 3 * cap ? 1 : 0);
    const LdsLaunch kl = pick_lds(dtype, hidden, n_layers, out_tiles, a.k1, a.embed_dim, a.rl != 0, light,
                                  rows / a.persistent_blocks);
    if (kl.k) {
      // one block per CU as long as there are wave tiles for them: a light
      // tick spreads its few tiles over every CU instead of filling a few
      const int rows = 32 * kl.rows;
      const int units = (a.n_total + rows - 1) / rows;
      const unsigned blocks = (unsigned)(units < a.persistent_blocks ? units : a.persistent_blocks);
      hipLaunchKernelGGL(kl.k, dim3(blocks), dim3(kl.waves * 64), 0, s, a);
      return hipGetLastError();
    }
  }
  if (a.persistent_blocks > 0) {
    RouteKernel ks = pick_stream(dtype, hidden, n_layers, out_tiles, a.k1, a.embed_dim, a.rl != 0);
    if (ks) {
      const int rows = kStreamWaves * 32;
      const int n_tiles = (a.n_total + rows - 1) / rows;
      const unsigned blocks = (unsigned)(n_tiles < a.persistent_blocks ? n_tiles : a.persistent_blocks);
      hipLaunchKernelGGL(ks, dim3(blocks), dim3(kStreamWaves * 64), 0, s, a);
      return hipGetLastError();
    }
  }
  if (dtype == IM_BF16) return launch_split(a, hidden, n_layers, out_tiles, !persistent, s);
  const F32Blocks f32 = f32_blocks(a.n_total, a.cus);
  const int nr = a.cus <= 0 || a.n_total <= 16 * a.cus ? 1 : 2;
  RouteKernel k = n_layers == 2 ? pick<2>(hidden, out_tiles, nr) : pick<3>(hidden, out_tiles, nr);
  RouteArgs f = a;
  f.pair_blocks = f32.pairs;
  unsigned blocks = (unsigned)(f32.pairs + f32.singles);
  if (hidden % 64 != 0) {
    blocks = (unsigned)((a.n_total + 63) / 64);   // 4 waves of 16 rows
  } else if (a.n_total_dev && nr == 2) {
    // Chain pools: whole rounds of blocks, which is the most that any row count up
    // to the bound takes. us per im_route, rows build included, blocks by the bound /
    // by the rows: 86 -> 256 -> 256 -> 15, 1,561 rows of at most 41,984, 26.3 / 20.2;
    // 405 -> 256 -> 256 -> 15, 1,711 rows of as many, 39.1 / 27.3.
    blocks = (unsigned)(a.cus * ((a.n_total - 1) / (32 * a.cus) + 1));
  }
  hipLaunchKernelGGL(k, dim3(blocks), dim3(256), 0, s, f);
  return hipGetLastError();
}

}  // namespace im

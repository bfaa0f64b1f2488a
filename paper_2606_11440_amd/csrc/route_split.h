// Route step, bf16 MLP policies of any shape: one block per group of rows, the
// output features of every hidden layer split over the block's waves.
//
// A block routes 32 NR rows. Its waves gather the rows' feature vectors into
// LDS as MFMA B fragments (the embedding by the LDS DMA path, 16 bytes a lane
// straight from the table; the tail features converted on the way), then each
// wave computes TPW 32-feature tiles of the layer for all the rows: a weight
// fragment is read once per block, from L2 into registers, and feeds NR MFMAs;
// an activation fragment is read from LDS and feeds TPW. A layer's output
// replaces its input in LDS (the accumulators hold it across the barrier). The
// output layer and the epilogue take one 32-row tile per wave.
//
// K ascends in every sum. With BL the bias is added to the finished sum; without,
// the sum starts from it, as in the persistent kernels, so that a shape that has
// one gets the same logits from both bit for bit. The two differ where an
// activation rounds to bf16 the other way (logits 1e-5 to 1e-4 apart, now and then
// an action), so a shape keeps the order it has: BL where it has no persistent
// kernel.
#pragma once
#include "route_dev.h"

namespace im {
namespace {

// Orders this wave's LDS accesses with the other waves' without waiting for
// its global loads in flight (weight fragments of the next layer).
__device__ __forceinline__ void lds_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0), vmcnt and expcnt at their maxima
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// acc[t][j] += W[T0 + t] h[j] over n K blocks whose activation fragments are in
// LDS (K block kb of row tile j at b[(kb NR + j) 64 + lane]) and whose weight
// fragments start at w + t * stride. D K blocks of weights are in flight.
template <int TPW, int NR, int D>
struct WeightRing {
  u32x4 r[D][TPW];
  const u32x4* p;   // this lane's fragments of the wave's first tile
  int stride;       // 16-byte words from one tile to the next
  int n;
  __device__ __forceinline__ u32x4 at(int kb, int t) const { return p[t * stride + kb * 64]; }
  __device__ __forceinline__ void start(const u32x4* w, int tile_stride, int kblocks) {
    p = w;
    stride = tile_stride;
    n = kblocks;
#pragma unroll
    for (int d = 0; d < D; ++d)
#pragma unroll
      for (int t = 0; t < TPW; ++t) r[d][t] = at(d < n ? d : n - 1, t);
  }
  __device__ __forceinline__ void run(const u32x4* b, f32x16 (&acc)[TPW][NR]) {
    for (int k0 = 0; k0 < n; k0 += D) {
#pragma unroll
      for (int d = 0; d < D; ++d) {
        const int kb = k0 + d;
        if (kb < n) {
          u32x4 x[NR];
#pragma unroll
          for (int j = 0; j < NR; ++j) x[j] = b[(kb * NR + j) * 64];
#pragma unroll
          for (int t = 0; t < TPW; ++t)
#pragma unroll
            for (int j = 0; j < NR; ++j) acc[t][j] = mfma_bf16(r[d][t], x[j], acc[t][j]);
          const int kn = kb + D < n ? kb + D : n - 1;
#pragma unroll
          for (int t = 0; t < TPW; ++t) r[d][t] = at(kn, t);
        }
      }
    }
  }
};

template <int H, int NL, int AT, int NR, int TPW, bool BL>
__global__ __launch_bounds__(H / 32 / TPW * 64, NR == 1 ? (AT == 3 && H < 512 ? 3 : 4) : (NR == 2 ? 3 : 2)) void route_bf16_split(RouteArgs a_in) {
  // chain pools: the tick's row count is on the device
  RouteArgs a = a_in;
  if (a_in.n_total_dev) a.n_total = min(*a_in.n_total_dev, a_in.n_total);   // the caller's buffers bound it
  constexpr int TH = H / 32, KH = H / 16, NW = TH / TPW, ROWS = 32 * NR;
  constexpr int KC = KH < 8 ? 8 : KH;         // K blocks of features in LDS at a time
  constexpr int D = TPW * NR >= 4 ? 4 : 8;    // weight fragments in flight per tile
  static_assert(TH % TPW == 0, "tiles split evenly over the waves");
  __shared__ u32x4 buf[KC * NR * 64];
  __shared__ int32_t s_e[ROWS], s_b[ROWS], s_bad[ROWS], s_id[ROWS];
  __shared__ uint64_t s_m[ROWS];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n = lane & 31, g = lane >> 5;
  const int32_t row0 = (int32_t)blockIdx.x * ROWS;
  if (row0 >= a.n_total) return;   // the whole block (chain pools' bound launch)

  // the first weight fragments and the biases travel with the row setup
  WeightRing<TPW, NR, D> ring;
  const int T0 = wave * TPW;
  const u32x4* W1 = (const u32x4*)a.W[0] + (size_t)T0 * a.k1 * 64 + lane;
  ring.start(W1, a.k1 * 64, a.k1 < KC ? a.k1 : KC);
  f32x16 acc[TPW][NR], bias[TPW];
  auto load_bias = [&](const float* b) {
#pragma unroll
    for (int t = 0; t < TPW; ++t) bias[t] = *(const f32x16*)(b + ((T0 + t) * 2 + g) * 16);
  };
  auto start_sums = [&]() {
#pragma unroll
    for (int t = 0; t < TPW; ++t)
#pragma unroll
      for (int j = 0; j < NR; ++j) acc[t][j] = BL ? f32x16{} : bias[t];
  };
  load_bias(a.bias[0]);

  const bool aligned = (a.embed_dim & 7) == 0 && ((uintptr_t)a.emb & 15) == 0;   // 16-byte aligned rows
  const int ke = aligned ? a.embed_dim / 16 : 0;   // K blocks that are all embedding
  int32_t q[NR];
#pragma unroll
  for (int j = 0; j < NR; ++j) {
    const int32_t v = a.q_idx[min(row0 + 32 * j + n, a.n_total - 1)];
    q[j] = v < 0 || (int64_t)v >= a.Q ? 0 : v;
  }
  // the embedding blocks [k0, k0 + kn) of the rows, straight into LDS
  auto gather_emb = [&](int k0, int kn) {
    for (int kb = wave; kb < kn && k0 + kb < ke; kb += NW) {
#pragma unroll
      for (int j = 0; j < NR; ++j) {
        const uint16_t* src = (const uint16_t*)a.emb + (size_t)q[j] * a.embed_dim + 16 * (k0 + kb) + 8 * g;
        __builtin_amdgcn_global_load_lds((const void*)src,
                                         (__attribute__((address_space(3))) void*)(buf + (kb * NR + j) * 64), 16, 0, 0);
      }
    }
  };
  // the other blocks of [k0, k0 + kn): load statistics, budget, padding (and an
  // embedding whose rows are not 16-byte aligned)
  auto gather_tail = [&](int k0, int kn) {
    const int t0 = ke > k0 ? ke - k0 : 0;
    for (int kb = t0 + wave; kb < kn; kb += NW) {
#pragma unroll
      for (int j = 0; j < NR; ++j) {
        RowCtx c;
        c.q = q[j];
        c.e = s_e[32 * j + n];
        c.budget = s_b[32 * j + n];
        buf[(kb * NR + j) * 64 + lane] = gather_bf16(a, c, k0 + kb, g);
      }
    }
  };
  gather_emb(0, a.k1 < KC ? a.k1 : KC);

  // ---- row contexts, one row per lane, while the embeddings travel ----
  for (int base = wave * 64; base < ROWS; base += NW * 64) {
    const int i = base + lane;
    const int32_t first = row0 + base;
    const int32_t last = min(row0 + min(base + 63, ROWS - 1), a.n_total - 1);
    int32_t e = 0, b = 0, bad = 0, id = -1;
    uint64_t m = 0;
    if (first <= last) {
      const int32_t rows[1] = {min(first + lane, last)};   // lanes past the rows repeat the last one
      b = a.budget[rows[0]];
      const int32_t qi = a.q_idx[rows[0]];
      int32_t env[1];
      find_envs<1>(a, first, last, rows, env);
      e = env[0];
      m = action_mask(a, e);
      if (a.rl && !a.greedy) id = a.ms[(size_t)e * a.M].next_id + (rows[0] - a.offsets[e]);
      bad = (qi < 0 || (int64_t)qi >= a.Q) ? IM_ERR_QIDX : 0;
    }
    if (i < ROWS) {
      s_e[i] = e;
      s_b[i] = b;
      s_bad[i] = bad;
      s_id[i] = id;
      s_m[i] = m;
    }
  }
  lds_barrier();

  // ---- layer 1 ----
  start_sums();
  for (int k0 = 0; k0 < a.k1; k0 += KC) {
    const int kn = a.k1 - k0 < KC ? a.k1 - k0 : KC;
    if (k0 != 0) {
      ring.start(W1 + k0 * 64, a.k1 * 64, kn);
      lds_barrier();   // every wave is done with the previous features
      gather_emb(k0, kn);
    }
    gather_tail(k0, kn);
    __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0): this wave's part of the features has landed
    lds_barrier();
    ring.run(buf + lane, acc);
  }

  auto store_frags = [&]() {
#pragma unroll
    for (int t = 0; t < TPW; ++t)
#pragma unroll
      for (int j = 0; j < NR; ++j) {
        u32x4 f0, f1;
        relu_to_frags(BL ? acc[t][j] + bias[t] : acc[t][j], f0, f1);
        buf[((2 * (T0 + t)) * NR + j) * 64 + lane] = f0;
        buf[((2 * (T0 + t) + 1) * NR + j) * 64 + lane] = f1;
      }
  };

  // ---- layer 2 ----
  if constexpr (NL == 3) {
    ring.start((const u32x4*)a.W[1] + (size_t)T0 * KH * 64 + lane, KH * 64, KH);
    lds_barrier();   // every wave is done reading the features
    store_frags();
    load_bias(a.bias[1]);
    start_sums();
    lds_barrier();
    ring.run(buf + lane, acc);
  }

  // ---- output layer and epilogue, a 32-row tile per wave ----
  WeightRing<AT, 1, 4> last;
  if (wave < NR) last.start((const u32x4*)a.W[NL - 1] + lane, KH * 64, KH);
  lds_barrier();   // every wave is done reading the layer's input
  store_frags();
  lds_barrier();
#pragma unroll 1
  for (int j = wave; j < NR; j += NW) {
    f32x16 out[AT], ob[AT];
#pragma unroll
    for (int T = 0; T < AT; ++T) {
      ob[T] = *(const f32x16*)(a.bias[NL - 1] + (T * 2 + g) * 16);
      out[T] = BL ? f32x16{} : ob[T];
    }
    if (j != wave) last.start((const u32x4*)a.W[NL - 1] + lane, KH * 64, KH);
    // this row tile's fragments are NR apart
    const u32x4* b = buf + j * 64 + lane;
#pragma unroll
    for (int k0 = 0; k0 < KH; k0 += 4) {
#pragma unroll
      for (int d = 0; d < 4 && d < KH; ++d) {
        const int kb = k0 + d;
        if (kb < KH) {
          const u32x4 x = b[kb * NR * 64];
#pragma unroll
          for (int T = 0; T < AT; ++T) out[T] = mfma_bf16(last.r[d][T], x, out[T]);
          if (kb + 4 < KH) {
#pragma unroll
            for (int T = 0; T < AT; ++T) last.r[d][T] = last.at(kb + 4, T);
          }
        }
      }
    }
    RowCtx r;
    const int i = 32 * j + n;
    r.r = row0 + i;
    r.live = r.r < a.n_total;
    r.e = s_e[i];
    r.q = 0;
    r.budget = s_b[i];
    r.bad = s_bad[i];
    r.id = s_id[i];
    r.amask = s_m[i];
    if constexpr (BL) {
#pragma unroll
      for (int T = 0; T < AT; ++T) out[T] += ob[T];
    }
    epilogue<AT>(r, out, g);
  }
}

typedef void (*RouteKernel)(RouteArgs);
struct SplitLaunch {
  RouteKernel k;
  int waves, rows;
};

template <int H, int NL, int AT, int NR, int TPW>
RouteKernel split_kernel(bool bias_last) {
  // the shapes (in part) that the persistent kernels cover
  if constexpr ((H == 256 && AT == 1) || (H == 512 && NL == 3 && AT >= 2)) {
    if (!bias_last) return route_bf16_split<H, NL, AT, NR, TPW, false>;
  }
  return route_bf16_split<H, NL, AT, NR, TPW, true>;
}
template <int H, int NL, int NR, int TPW>
SplitLaunch pick_at(int at, bool bias_last) {
  RouteKernel k = at == 1 ? split_kernel<H, NL, 1, NR, TPW>(bias_last)
                          : (at == 2 ? split_kernel<H, NL, 2, NR, TPW>(bias_last) : split_kernel<H, NL, 3, NR, TPW>(bias_last));
  return {k, H / 32 / TPW, 32 * NR};
}
template <int H, int NL>
SplitLaunch pick_rows(int at, bool bias_last, int size) {
  if (size == 0 || H == 32) return pick_at<H, NL, 1, 1>(at, bias_last);   // hidden 32: one wave a block
  if constexpr (H >= 256) {
    if (size == 2) return pick_at<H, NL, 4, 2>(at, bias_last);
  }
  if constexpr (H > 32) return pick_at<H, NL, 2, H == 512 ? 2 : 1>(at, bias_last);
}
template <int H>
SplitLaunch pick_nl(int nl, int at, bool bias_last, int size) {
  return nl == 2 ? pick_rows<H, 2>(at, bias_last, size) : pick_rows<H, 3>(at, bias_last, size);
}

bool split_supported(int hidden) {
  return hidden == 32 || hidden == 64 || hidden == 128 || hidden == 256 || hidden == 512;
}

// Rows per block. Up to one 32-row block per compute unit the launch is bound
// by one block's latency, which grows with its rows; up to one 64-row block
// per compute unit a second round of blocks costs more than the second row
// tile. Past that the wide layers (hidden 256, 512) take 128 rows and two
// feature tiles per wave, which halves the weight bytes from L2 and the
// activation bytes from LDS per MFMA; the narrow ones, whose weights stay in
// the vector cache, keep 64 rows (more blocks per compute unit): at hidden 128
// the 128-row shape is ahead in a band around 131,072 rows only. us per launch at
// 32 / 64 / 128 rows per block, greedy (128 rows of the narrow shapes: compiled for
// the comparison):
//   405 -> 256 -> 256 -> 15  8,192 rows 10.0 / 12.2 / 17.2, 16,384 rows 14.5 / 12.5 / 17.3,
//                            65,536 rows 50.8 / 36.0 / 30.6, 131,072 rows 97.6 / 68.1 / 57.3
//   97 -> 128 -> 128 -> 32   8,192 rows 5.2 / 6.0 / 10.3, 65,536 rows 14.4 / 10.5 / 12.6,
//                            131,072 rows 25.9 / 18.4 / 16.3, 262,144 rows 53.7 / 35.1 / 37.6
//   85 -> 64 -> 15           8,192 rows 4.5 / 4.9 / 10.6, 131,072 rows 12.4 / 9.4 / 13.5
// bias_last: the shape has no persistent kernel.
hipError_t launch_split(const RouteArgs& a, int hidden, int n_layers, int out_tiles, bool bias_last, hipStream_t s) {
  const int64_t cus = a.persistent_blocks > 0 ? a.persistent_blocks : a.cus;
  const int size = a.n_total <= 32 * cus ? 0 : (a.n_total <= 64 * cus ? 1 : 2);
  SplitLaunch l{};
  switch (hidden) {
    case 32: l = pick_nl<32>(n_layers, out_tiles, bias_last, size); break;
    case 64: l = pick_nl<64>(n_layers, out_tiles, bias_last, size); break;
    case 128: l = pick_nl<128>(n_layers, out_tiles, bias_last, size); break;
    case 256: l = pick_nl<256>(n_layers, out_tiles, bias_last, size); break;
    case 512: l = pick_nl<512>(n_layers, out_tiles, bias_last, size); break;
    default: return hipErrorInvalidValue;
  }
  const unsigned blocks = (unsigned)(((int64_t)a.n_total + l.rows - 1) / l.rows);
  hipLaunchKernelGGL(l.k, dim3(blocks), dim3(l.waves * 64), 0, s, a);
  return hipGetLastError();
}

}  // namespace
}  // namespace im

// Device code shared by the route kernels: row contexts (env lookup, action
// mask, feature gather), bf16 packing, the masked argmax / RL-rollout epilogue
// and the LDS DMA of one weight fragment.
#pragma once
#include <math.h>

#include "im_internal.h"
#include "wave.h"

namespace im {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f32x16 mfma_bf16(u32x4 a, u32x4 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a),
                                                 __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}
typedef float f32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ f32x4 mfma16_f32(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

struct RowCtx {
  int32_t r;        // request row (tail lanes: >= n_total)
  bool live;        // r < n_total
  int32_t bad;      // error bits of the row (IM_ERR_QIDX, IM_ERR_ROLE); 0 when valid
  int32_t e;        // env of the row
  int32_t q;        // embedding row (0 when bad)
  int32_t budget;
  uint64_t amask;   // bit a set when action a is valid
  int32_t id = -1;  // the row's request id where the setup already read it (RL sampling)
};

// Valid actions of env e: bit a set when model a / K is valid in the env's
// snapshot row (enabled, c_m > 0, queue below capacity).
// The M <= 32 validity bytes start 16-byte aligned (byte 16 M of a row whose
// stride is a multiple of 32 bytes) and the row's padding covers two 16-byte
// words from there, so they arrive in one or two independent loads (a byte
// loop would wait for each byte in turn).
__device__ __forceinline__ uint32_t nonzero_bytes(uint32_t x) {
  // bit i of the result: byte i of x is nonzero (OR-fold each byte into its
  // low bit, then gather bits 0, 8, 16, 24 with one multiply: the shifted
  // copies land on distinct bits, so no carries)
  x |= x >> 4;
  x |= x >> 2;
  x |= x >> 1;
  return ((x & 0x01010101u) * 0x00204081u) >> 21 & 0xfu;
}
__device__ __forceinline__ uint32_t valid_models16(const u32x4 w) {
  return nonzero_bytes(w.x) | nonzero_bytes(w.y) << 4 | nonzero_bytes(w.z) << 8 | nonzero_bytes(w.w) << 12;
}
// The raw validity words of env e (both loaded for every M: the row's padding
// covers them) and the action mask computed from them once they have arrived.
struct ValidRaw {
  u32x4 w0, w1;
};
__device__ __forceinline__ ValidRaw load_valid(const RouteArgs& a, int e) {
  const u32x4* v = (const u32x4*)(a.snap + (size_t)e * snap_stride(a.M) + snap_valid_offset(a.M));
  return {v[0], v[1]};
}
__device__ __forceinline__ uint64_t mask_of(const RouteArgs& a, const ValidRaw& v) {
  uint32_t vm = valid_models16(v.w0);
  if (a.M > 16) vm |= valid_models16(v.w1) << 16;
  if (a.M < 32) vm &= (1u << a.M) - 1u;   // bytes past the M-th are padding
  const uint64_t kmask = (a.K >= 64) ? ~0ull : ((1ull << a.K) - 1ull);
  uint64_t am = 0;
  for (int m = 0; m < a.M; ++m)
    if ((vm >> m) & 1u) am |= kmask << (m * a.K);
  return am;
}
__device__ __forceinline__ uint64_t action_mask(const RouteArgs& a, int e) { return mask_of(a, load_valid(a, e)); }

// Env of rows r[] (per lane) for a wave whose rows lie in [rfirst, rlast]:
// one coalesced load of a 64-entry window of offsets around an interpolated
// guess; a uniform binary search when the guess misses.
__device__ __forceinline__ int32_t find_env_bsearch(const RouteArgs& a, int32_t r) {
  int lo = 0, hi = a.E;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (a.offsets[mid] <= r) lo = mid; else hi = mid - 1;
  }
  return lo < a.E ? lo : a.E - 1;
}

// First guess of the env window of rows from rfirst on, and its offsets
// (lane i: offsets[e_lo + i]); find_envs_in completes the lookup.
struct EnvWindow {
  int32_t e_lo, ow;
};
__device__ __forceinline__ EnvWindow env_window(const RouteArgs& a, int32_t rfirst) {
  EnvWindow w;
  int32_t e_lo = (int32_t)((float)rfirst * a.envs_per_row) - 16;
  w.e_lo = e_lo < 0 ? 0 : (e_lo > a.E - 1 ? a.E - 1 : e_lo);
  const int32_t wi = w.e_lo + lane_id();
  w.ow = a.offsets[wi < a.E ? wi : a.E];
  return w;
}

template <int NR>
__device__ __forceinline__ void find_envs_in(const RouteArgs& a, EnvWindow w, int32_t rfirst, int32_t rlast,
                                             const int32_t (&r)[NR], int32_t (&e)[NR]) {
  const int lane = lane_id();
  int32_t e_lo = w.e_lo;
  int32_t wi;
  int32_t ow = w.ow;
  bool ok = __builtin_amdgcn_readfirstlane(ow) <= rfirst &&
            rlast < __builtin_amdgcn_readlane(ow, 63);
  if (!ok) {
    e_lo = find_env_bsearch(a, rfirst);
    wi = e_lo + lane;
    ow = a.offsets[wi < a.E ? wi : a.E];
    ok = rlast < __builtin_amdgcn_readlane(ow, 63);
  }
  if (ok) {
    // The window's offsets are ascending. The env of row x is e_lo - 1 plus
    // the number of window offsets <= x: those <= rfirst (one ballot), plus
    // the env boundaries inside the wave's rows (rfirst, rlast], few per wave.
    const int base = e_lo - 1 + popc64(ballot(ow <= rfirst));
#pragma unroll
    for (int j = 0; j < NR; ++j) e[j] = base;
    uint64_t bnd = ballot(ow > rfirst && ow <= rlast);
    while (bnd) {
      const int b = __builtin_ctzll(bnd);
      bnd &= bnd - 1;
      const int32_t ob = __builtin_amdgcn_readlane(ow, b);
#pragma unroll
      for (int j = 0; j < NR; ++j) e[j] += ob <= r[j] ? 1 : 0;
    }
  } else {
#pragma unroll
    for (int j = 0; j < NR; ++j) e[j] = find_env_bsearch(a, r[j] < a.n_total ? r[j] : a.n_total - 1);
  }
#pragma unroll
  for (int j = 0; j < NR; ++j) e[j] = e[j] < 0 ? 0 : (e[j] > a.E - 1 ? a.E - 1 : e[j]);
}

template <int NR>
__device__ __forceinline__ void find_envs(const RouteArgs& a, int32_t rfirst, int32_t rlast,
                                          const int32_t (&r)[NR], int32_t (&e)[NR]) {
  find_envs_in<NR>(a, env_window(a, rfirst), rfirst, rlast, r, e);
}

// Row context of row r in env e from its already loaded record fields.
__device__ __forceinline__ RowCtx row_ctx_from(const RouteArgs& a, int32_t r, int32_t e, int32_t q,
                                               int32_t budget) {
  RowCtx c;
  c.r = r;
  c.live = r < a.n_total;
  c.e = e;
  c.bad = (q < 0 || (int64_t)q >= a.Q) ? IM_ERR_QIDX : 0;
  c.q = c.bad ? 0 : q;
  c.budget = budget;
  c.amask = 0;   // set by the caller from load_valid / mask_of
  return c;
}

__device__ __forceinline__ RowCtx row_setup_env(const RouteArgs& a, int32_t r, int32_t e) {
  RowCtx c;
  c.r = r;
  c.live = r < a.n_total;
  const int32_t rr = c.live ? r : a.n_total - 1;
  c.e = e;
  const int32_t q = a.q_idx[rr];
  c.bad = (q < 0 || (int64_t)q >= a.Q) ? IM_ERR_QIDX : 0;
  c.q = c.bad ? 0 : q;
  c.budget = a.budget[rr];
  c.amask = action_mask(a, e);
  return c;
}

// The same, leaving the action mask to the caller (load_valid's words are in
// flight with the row's q_idx and budget).
__device__ __forceinline__ RowCtx row_setup_env_raw(const RouteArgs& a, int32_t r, int32_t e, ValidRaw& vr) {
  RowCtx c;
  c.r = r;
  c.live = r < a.n_total;
  const int32_t rr = c.live ? r : a.n_total - 1;
  c.e = e;
  const int32_t q = a.q_idx[rr];
  c.bad = (q < 0 || (int64_t)q >= a.Q) ? IM_ERR_QIDX : 0;
  c.q = c.bad ? 0 : q;
  c.budget = a.budget[rr];
  vr = load_valid(a, e);
  c.amask = 0;   // mask_of(a, vr) once the words have arrived
  return c;
}

// Feature k >= embed_dim of a row: the env's load statistics (stat-major:
// queue depth of all models, busy/c_m, latency EWMA, backlog; read from the
// snapshot row), then the normalised budget, then zeros.
__device__ __forceinline__ float tail_feature(const RouteArgs& a, const RowCtx& c, int k) {
  const int k2 = k - a.embed_dim;
  if (k2 < 4 * a.M) return a.snap[(size_t)c.e * snap_stride(a.M) + k2];
  if (k2 == 4 * a.M) return (float)c.budget * a.inv_bud;
  return 0.f;
}

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

// Two fp32 values to packed bf16 (round to nearest even), one
// v_cvt_pk_bf16_f32; element 0 in the low half.
__device__ __forceinline__ uint32_t pack2(float lo, float hi) {
  const f32x2 v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

// ReLU of a float as one integer max on its bits: every negative value
// (and -0) has the sign bit set, so it is below 0 as an int32.
__device__ __forceinline__ float relu(float x) {
  return __int_as_float(max(__float_as_int(x), 0));
}

// bf16(ReLU(lo)), bf16(ReLU(hi)) packed. Rounding to nearest even keeps the
// sign (a negative value rounds to a negative value or -0), so the ReLU is
// applied after rounding, to both halves at once, as a packed signed 16-bit
// max with 0.
__device__ __forceinline__ uint32_t relu_pack2(float lo, float hi) {
  typedef short s16x2 __attribute__((ext_vector_type(2)));
  const s16x2 r = __builtin_bit_cast(s16x2, pack2(lo, hi));
  return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(r, (s16x2){0, 0}));
}

// Layer-1 B fragment of K block kb (bf16): features 16 kb + 8 g + j, j = 0..7.
__device__ __forceinline__ u32x4 gather_bf16(const RouteArgs& a, const RowCtx& c, int kb, int g) {
  const int k0 = 16 * kb + 8 * g;
  const uint16_t* emb = (const uint16_t*)a.emb;
  const bool aligned = (a.embed_dim & 7) == 0;
  if (aligned && k0 + 8 <= a.embed_dim)
    return *(const u32x4*)(emb + (size_t)c.q * a.embed_dim + k0);
  float f[8];
  if (aligned && k0 >= a.embed_dim) {
    // 8 tail features: two aligned float4 loads of the snapshot row, then
    // the budget feature and zero padding selected by index.
    // The row is read only when the block holds a load statistic (k2 < 4M):
    // the 8 floats from k2 then lie inside the row's stride (>= 4M + 9).
    const int k2 = k0 - a.embed_dim;
    float4 lo = make_float4(0.f, 0.f, 0.f, 0.f), hi = lo;
    if (k2 < 4 * a.M) {
      const float* row = a.snap + (size_t)c.e * snap_stride(a.M) + k2;
      lo = *(const float4*)row;
      hi = *(const float4*)(row + 4);
    }
    const float v[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
    const float fb = (float)c.budget * a.inv_bud;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int kk = k2 + j;
      f[j] = kk < 4 * a.M ? v[j] : (kk == 4 * a.M ? fb : 0.f);
    }
  } else {
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int k = k0 + j;
      f[j] = k < a.embed_dim ? bf16_to_f32(emb[(size_t)c.q * a.embed_dim + k])
                             : tail_feature(a, c, k);
    }
  }
  u32x4 v;
  v.x = pack2(f[0], f[1]);
  v.y = pack2(f[2], f[3]);
  v.z = pack2(f[4], f[5]);
  v.w = pack2(f[6], f[7]);
  return v;
}

// Layer-1 B fragments of a row in two steps, so that a wave tile's gather is
// one round trip: gather_issue loads every embedding word and the raw
// snapshot words of the tail blocks (the load statistics; a lane whose block
// starts past them reads from the row's last statistic on, which stays inside
// the row, and ignores the words), gather_finish converts the tail blocks once
// they have arrived (the arithmetic of gather_ct).
template <int ED, int KB1>
struct TailRaw {
  static constexpr int KE = ED / 16 < KB1 ? ED / 16 : KB1;   // K blocks inside the embedding
  static constexpr int KT = KB1 - KE;                          // tail blocks
  float4 t[KT > 0 ? KT : 1][2];
};
template <int ED, int KB1>
__device__ __forceinline__ void gather_issue(const RouteArgs& a, const RowCtx& c, int g, u32x4 (&x)[KB1],
                                             TailRaw<ED, KB1>& raw) {
  static_assert(ED % 16 == 0, "embedding width must be a multiple of 16");
  using TR = TailRaw<ED, KB1>;
  const uint16_t* emb = (const uint16_t*)a.emb;
#pragma unroll
  for (int kb = 0; kb < TR::KE; ++kb) x[kb] = *(const u32x4*)(emb + (size_t)c.q * ED + 16 * kb + 8 * g);
  const int n4 = 4 * a.M;
#pragma unroll
  for (int t = 0; t < TR::KT; ++t) {
    const int k2 = 16 * t + 8 * g;
    const float* row = a.snap + (size_t)c.e * snap_stride(a.M) + (k2 < n4 ? k2 : n4 - 1);
    raw.t[t][0] = *(const float4*)row;
    raw.t[t][1] = *(const float4*)(row + 4);
  }
}
template <int ED, int KB1>
__device__ __forceinline__ void gather_finish(const RouteArgs& a, const RowCtx& c, int g, u32x4 (&x)[KB1],
                                              const TailRaw<ED, KB1>& raw) {
  using TR = TailRaw<ED, KB1>;
  const int n4 = 4 * a.M;
  const float fb = (float)c.budget * a.inv_bud;
#pragma unroll
  for (int t = 0; t < TR::KT; ++t) {
    const int k2 = 16 * t + 8 * g;
    const float4 lo = raw.t[t][0], hi = raw.t[t][1];
    const float v[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
    float f[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int kk = k2 + i;
      f[i] = kk < n4 ? v[i] : (kk == n4 ? fb : 0.f);
    }
    u32x4 r;
    r.x = pack2(f[0], f[1]);
    r.y = pack2(f[2], f[3]);
    r.z = pack2(f[4], f[5]);
    r.w = pack2(f[6], f[7]);
    x[TR::KE + t] = r;
  }
}

// Philox4x32-10 block (Salmon, Moraes, Dror, Shaw, SC 2011): ten rounds of
// two 32x32 -> 64-bit products by the round multipliers, whose high halves are
// xored with the other two counter words and the key; the key advances by the
// Weyl constants after every round.
__device__ __forceinline__ uint4 philox10(uint4 c, uint32_t k0, uint32_t k1) {
#pragma unroll
  for (int i = 0; i < 10; ++i) {
    // one 32x32 -> 64-bit product each (a single v_mad_u64_u32)
    const uint64_t p0 = (uint64_t)0xD2511F53u * c.x;
    const uint64_t p1 = (uint64_t)0xCD9E8D57u * c.z;
    c = make_uint4((uint32_t)(p1 >> 32) ^ c.y ^ k0, (uint32_t)p1, (uint32_t)(p0 >> 32) ^ c.w ^ k1,
                   (uint32_t)p0);
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
  }
  return c;
}

// Exponential variate E = -ln U of a 32-bit word, U = (top 23 bits + 1/2)
// 2^-23 (exact in fp32). Above U = 15/16, 1 - U = d is exact and -ln(1 - d)
// is summed as d + d^2/2 + ... + d^7/7 (the rest is below 2^-24 d), so E keeps
// its relative precision however close U is to 1.
__device__ __forceinline__ float expo_of(uint32_t w) {
  const uint32_t k = w >> 9;
  const float u = ((float)k + 0.5f) * (1.0f / 8388608.0f);
  const float d = ((float)(8388608u - k) - 0.5f) * (1.0f / 8388608.0f);
  const float series =
      d * (1.f + d * (0.5f + d * (1.f / 3.f + d * (0.25f + d * (0.2f + d * (1.f / 6.f + d * (1.f / 7.f)))))));
  return d < 0.0625f ? series : -__logf(u);
}

// Request id of a row: its env's next id plus the row's position in the env.
__device__ __forceinline__ uint32_t request_id(const RouteArgs& a, const RowCtx& c) {
  const int32_t rr = c.live ? c.r : a.n_total - 1;
  return (uint32_t)(a.ms[(size_t)c.e * a.M].next_id + (rr - a.offsets[c.e]));
}

// RL-rollout outputs of one row from its logits (lane pair n, n + 32 holds
// the row's actions 32 T + 8 (v / 4) + 4 g + v % 4): pi is the softmax of
// the logits over the valid actions, shifted by their largest logit `zmax`
// (action `amax`, -1 when none is valid); the action is the Gumbel-max draw
// (or `amax` when greedy), its log-probability z_a - logsumexp, the entropy
// logsumexp - sum pi z, and the value head's row A. The Gumbel-max draw
// argmax z_a - ln(E_a), E_a = -ln U_a, is taken as the equivalent argmax of
// exp(z_a - zmax) / E_a (one logarithm per action instead of two).
template <int AT>
__device__ __forceinline__ void rl_outputs(const RouteArgs& a, const RowCtx& c,
                                           const f32x16 (&acc)[AT], int g, float zmax, int amax) {
  const bool sample = a.greedy == 0;
  uint32_t id = 0;
  if (sample) {
    id = c.id >= 0 ? (uint32_t)c.id : request_id(a, c);
  }
  float s = 0.f, sz = 0.f, val = 0.f, bs = 0.f, bz = 0.f;
  int bsa = -1;
#pragma unroll
  for (int T = 0; T < AT; ++T) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int a0 = 32 * T + 8 * j + 4 * g;   // this lane's 4 consecutive actions: one Philox block
      uint4 w = make_uint4(0, 0, 0, 0);
      if (sample && a0 < a.A) w = philox10(make_uint4(id, (uint32_t)c.e, (uint32_t)(a0 >> 2), 0u), a.seed_lo, a.seed_hi);
      const uint32_t wv[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int act = a0 + i;
        const float z = acc[T][4 * j + i];
        if (act == a.A) val = z;
        if (act < a.A && ((c.amask >> act) & 1ull)) {
          const float ex = __expf(z - zmax);
          s += ex;
          sz += ex * z;
          const float sc = sample ? __fdividef(ex, expo_of(wv[i])) : z;
          if (bsa < 0 || sc > bs) { bs = sc; bsa = act; bz = z; }   // actions ascend: ties keep the lowest
        }
      }
    }
  }
  s += __shfl_xor(s, 32, 64);
  sz += __shfl_xor(sz, 32, 64);
  val += __shfl_xor(val, 32, 64);                  // one lane of the pair holds row A
  const float obs = __shfl_xor(bs, 32, 64), obz = __shfl_xor(bz, 32, 64);
  const int obsa = __shfl_xor(bsa, 32, 64);
  if (obsa >= 0 && (bsa < 0 || obs > bs || (obs == bs && obsa < bsa))) { bs = obs; bsa = obsa; bz = obz; }
  if (!c.live || g != 0) return;
  const bool any = amax >= 0 && !c.bad;
  const float lse = any ? zmax + __logf(s) : 0.f;
  a.actions[c.r] = any ? bsa : -1;
  if (c.bad) atomicOr(a.err, c.bad);
  if (a.logp) a.logp[c.r] = any ? bz - lse : 0.f;
  if (a.entropy) a.entropy[c.r] = any ? lse - sz / s : 0.f;
  if (a.value) a.value[c.r] = c.bad ? 0.f : val;
}

// Masked argmax over the lane pair (n, n + 32), logits store, action store
// (or the RL-rollout outputs). RL: 0 = greedy route only, 1 = RL outputs
// only, 2 = either, chosen by a.rl at run time.
template <int AT, int RL = 2>
__device__ __forceinline__ void epilogue(const RouteArgs& a, const RowCtx& c, f32x16 (&acc)[AT],
                                         const float* bias, int g) {
  float best = 0.f;
  int ba = -1;
#pragma unroll
  for (int T = 0; T < AT; ++T) {
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int act = 32 * T + 8 * (v >> 2) + 4 * g + (v & 3);
      const float z = bias ? acc[T][v] + bias[(T * 2 + g) * 16 + v] : acc[T][v];
      acc[T][v] = z;
      if (act < a.A && ((c.amask >> act) & 1ull)) {
        if (ba < 0 || z > best) { best = z; ba = act; }
      }
    }
  }
  const float ob = __shfl_xor(best, 32, 64);
  const int oa = __shfl_xor(ba, 32, 64);
  if (oa >= 0 && (ba < 0 || ob > best || (ob == best && oa < ba))) { best = ob; ba = oa; }
  if (RL == 1 || (RL == 2 && a.rl)) {
    rl_outputs<AT>(a, c, acc, g, best, ba);
  } else if (c.live && g == 0) {
    a.actions[c.r] = c.bad ? -1 : ba;
    if (c.bad) atomicOr(a.err, c.bad);
  }
  if (!c.live) return;
  if (a.logits) {
    float* out = a.logits + (size_t)c.r * a.A;
#pragma unroll
    for (int T = 0; T < AT; ++T) {
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int act = 32 * T + 8 * (v >> 2) + 4 * g + (v & 3);
        if (act < a.A) out[act] = c.bad ? 0.f : acc[T][v];
      }
    }
  }
}

// ReLU + bf16 rounding of one accumulator tile (bias already included).
__device__ __forceinline__ void relu_to_frags(const f32x16& acc, u32x4& f0, u32x4& f1) {
  f0.x = relu_pack2(acc[0], acc[1]);   f0.y = relu_pack2(acc[2], acc[3]);
  f0.z = relu_pack2(acc[4], acc[5]);   f0.w = relu_pack2(acc[6], acc[7]);
  f1.x = relu_pack2(acc[8], acc[9]);   f1.y = relu_pack2(acc[10], acc[11]);
  f1.z = relu_pack2(acc[12], acc[13]); f1.w = relu_pack2(acc[14], acc[15]);
}

// One 1 KB fragment (64 lanes x 16 B) from global memory into LDS; `dst` is
// wave-uniform, lane l's 16 bytes land at dst + 16 l.
__device__ __forceinline__ void dma_frag(u32x4* dst, const u32x4* src, int lane) {
  __builtin_amdgcn_global_load_lds((const void*)(src + lane),
                                   (__attribute__((address_space(3))) void*)dst, 16, 0, 0);
}

}  // namespace
}  // namespace im

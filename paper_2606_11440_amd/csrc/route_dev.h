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

// Valid actions of env e: bit a set when action a's model is valid (enabled,
// c_m > 0, queue below capacity), kept ready in the env's snapshot row.
__device__ __forceinline__ uint64_t action_mask(const RouteArgs& a, int e) {
  return *(const uint64_t*)(a.snap + (size_t)e * snap_stride(a.M) + snap_mask_offset(a.M));
}

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
  c.amask = action_mask(a, e);
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
    // the 8 floats from k2 then lie inside the row's stride (>= 4M + 8).
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
// they have arrived.
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

// The kernel's arguments (every route kernel takes one RouteArgs) where the
// runtime put them, for code after a wave's matrix work: read there again with
// scalar loads, they need not stay in scalar registers through it (the RL
// kernels spilled them into vector registers). Chain pools: n_total is the bound.
typedef const __attribute__((address_space(4))) RouteArgs* KernArgs;
__device__ __forceinline__ KernArgs late_args() {
  KernArgs k = (KernArgs)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(k));
  return k;
}

// Request id of a row: its env's next id plus the row's position in the env
// (a row past the last one: a number nobody uses).
__device__ __forceinline__ uint32_t request_id(KernArgs a, const RowCtx& c) {
  return (uint32_t)(a->ms[(size_t)c.e * a->M].next_id + (c.r - a->offsets[c.e]));
}

// All ones where bit `bit` of `w` is set, else 0.
__device__ __forceinline__ uint32_t bit_ones(uint32_t w, int bit) {
  return (uint32_t)__builtin_amdgcn_sbfe((int)w, (uint32_t)bit, 1u);
}
// A logit, or `low` (-inf) when `masked` is all ones (one v_bfi_b32).
__device__ __forceinline__ float mask_logit(float z, uint32_t masked, uint32_t low) {
  return __uint_as_float((low & masked) | (__float_as_uint(z) & ~masked));
}
// -inf in a register of the code around, not in one kept through the kernel's loop.
constexpr uint32_t kMinusInf = 0xff800000u;
__device__ __forceinline__ uint32_t minus_inf() {
  uint32_t low = kMinusInf;
  asm volatile("" : "+s"(low));
  return low;
}
// Largest operand, NaN if one of them is.
__device__ __forceinline__ float maximum3(float x, float y, float z) {
  float r;
  asm("v_maximum3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(x), "v"(y), "v"(z));
  return r;
}
// Largest operand that is not NaN (one instruction; fmaxf would first
// canonicalise each operand).
__device__ __forceinline__ float max3(float x, float y, float z) {
  float r;
  asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(x), "v"(y), "v"(z));
  return r;
}
__device__ __forceinline__ int32_t as_int(float x) { return __float_as_int(x); }

// Softmax sums and the Gumbel-max draw over the actions a lane holds, four
// consecutive ones (a Philox block) at a time. pi is the softmax of the logits
// over the valid actions, shifted by their largest logit zmax. The draw argmax
// z_a - ln(E_a), E_a = -ln U_a, is taken as the equivalent argmax of
// exp(z_a - zmax) / -log2(U_a): one logarithm and one reciprocal per action,
// and ln 2 scales every score alike. U_a = (top 23 bits + 1/2) 2^-23 is exact
// in fp32, and the hardware log2 keeps its relative precision up to U = 1 - 2^-24.
// Over all 2^23 values of U a score exp / -log2(U) is at most 2.0e-7 off (5.8e-8
// rms; the logarithm alone 1.2e-7); a series or logf for -ln U and a full division
// gave 2.4e-7 (6.1e-8). Branch-free: a masked action has exp 0 and logit 0 in the
// sums, and a score of 0 never exceeds the best.
struct RlSums {
  float s = 0.f, sz = 0.f;    // sum of exp(z - zmax), of exp(z - zmax) z
  float bs = 0.f, bz = 0.f;   // best score, its logit
  int32_t ba = 127;           // its action
};
template <bool SAMPLE>
__device__ __forceinline__ void rl_block(RlSums& r, const float (&z)[4], uint32_t masked_bits, float zmax,
                                         int act0, uint4 w) {
  const uint32_t wv[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const uint32_t on = ~bit_ones(masked_bits, i);
    const float ex = __uint_as_float(__float_as_uint(__builtin_amdgcn_exp2f((z[i] - zmax) * 1.44269504088896341f)) & on);
    const float zv = __uint_as_float(__float_as_uint(z[i]) & on);
    r.s += ex;
    r.sz = fmaf(ex, zv, r.sz);
    if constexpr (SAMPLE) {
      const float u = fmaf((float)(wv[i] >> 9), 1.0f / 8388608.0f, 0.5f / 8388608.0f);
      const float sc = ex * __builtin_amdgcn_rcpf(-__builtin_amdgcn_logf(u));
      const bool take = sc > r.bs;   // actions ascend: ties keep the lowest
      r.bs = take ? sc : r.bs;
      r.bz = take ? zv : r.bz;
      r.ba = take ? act0 + i : r.ba;
    }
  }
}
// Adds the sums of another lane of the same row; the larger score wins, the
// lower action on a tie.
__device__ __forceinline__ void rl_join(RlSums& r, float s, float sz, float bs, float bz, int32_t ba) {
  r.s += s;
  r.sz += sz;
  const bool take = bs > r.bs || (bs == r.bs && ba < r.ba);
  r.bs = take ? bs : r.bs;
  r.bz = take ? bz : r.bz;
  r.ba = take ? ba : r.ba;
}
// The outputs of row c: any: some action is valid and the row's inputs are.
__device__ __forceinline__ void rl_store(KernArgs a, const RowCtx& c, RlSums& r, float zmax, int32_t amax,
                                         float val) {
  const bool any = c.amask != 0 && !c.bad;
  if (a->greedy) {
    r.ba = amax;
    r.bz = zmax;
  } else if (r.ba >= 64) {
    r.ba = __ffsll((unsigned long long)c.amask) - 1;   // no score above 0 (logits that are not finite)
  }
  const float lse = zmax + __logf(r.s);
  a->actions[c.r] = any ? r.ba : -1;
  if (c.bad) atomicOr(a->err, c.bad);
  if (a->logp) a->logp[c.r] = any ? r.bz - lse : 0.f;
  if (a->entropy) a->entropy[c.r] = any ? lse - r.sz / r.s : 0.f;
  if (a->value) a->value[c.r] = c.bad ? 0.f : val;
}

// Stores the four consecutive logits act .. act + 3 of a row, those below A.
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
__device__ __forceinline__ void store_logits(KernArgs a, float* row, int act, float z0, float z1, float z2,
                                             float z3) {
  if (act + 4 <= a->A) {
    *(f32x4u*)(row + act) = (f32x4u){z0, z1, z2, z3};
  } else {
    if (act < a->A) row[act] = z0;
    if (act + 1 < a->A) row[act + 1] = z1;
    if (act + 2 < a->A) row[act + 2] = z2;
  }
}

// bit 32 T + 8 j + i of the words: action 32 T + 8 j + 4 g + i is masked
struct MaskWords {
  uint32_t w[2];
};
__device__ __forceinline__ MaskWords mask_words(uint64_t am, int g) {
  const uint64_t inv = (uint64_t)((int64_t)~am >> (4 * g));
  return {{(uint32_t)inv, (uint32_t)(inv >> 32)}};
}
constexpr int action_tiles(int at) { return at < 2 ? at : 2; }   // at most 64 actions; a third tile holds the value row only

// The argmax is that of a scan over the valid actions which takes each one whose
// logit exceeds the best one's: a NaN is passed over, unless the lowest valid
// action's logit is NaN, which nothing exceeds. NaN is rare and dealt with after
// the fact: where a row has one among its valid logits, this finds whether it is
// the lowest valid action's and, with ARGMAX, the argmax of the others (both lanes
// of the pair).
struct NanScan {
  bool first_nan;
  int32_t ba;   // lowest action of the largest logit that is not NaN (where that is above -inf)
  float best;   // that logit
};
template <int AT, bool ARGMAX>
__device__ __forceinline__ NanScan nan_scan(uint64_t am, const f32x16 (&acc)[AT], int g) {
  asm volatile("" : "+v"(am));   // the masked logits are formed again, not kept for this
  const MaskWords mw = mask_words(am, g);
  const int first = __ffsll((unsigned long long)am) - 1 - 4 * g;
  const uint32_t low = minus_inf();
  float best = __uint_as_float(low);
  int32_t nan = 0, ba = 127;
#pragma unroll
  for (int T = 0; T < action_tiles(AT); ++T)
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int act = 32 * T + 8 * (v >> 2) + (v & 3);
      const float z = mask_logit(acc[T][v], bit_ones(mw.w[T], 8 * (v >> 2) + (v & 3)), low);
      nan |= first == act && z != z;
      if constexpr (ARGMAX) {
        ba = z > best ? act : ba;
        best = max3(best, z, z);
      }
    }
  nan |= xshfl<32>(nan);
  if constexpr (!ARGMAX) return {nan != 0, 127, 0.f};
  ba += 4 * g;
  int32_t x, y;
  swap_halves<32>(as_int(best), x, y);
  const float all = max3(__int_as_float(x), __int_as_float(y), __int_as_float(y));
  ba = best == all ? ba : 127;
  swap_halves<32>(ba, x, y);
  return {nan != 0, x < y ? x : y, all};
}

// One 32-row tile's part of the outputs: lane (n, g) holds the actions 32 T +
// 8 (v / 4) + 4 g + v % 4 of its row n. `am` is the row's action mask, `id` and
// `e` its request id and env (RL sampling). best: the row's largest valid logit
// (both lanes of the pair): NaN is passed over with RL outputs, where the sum of
// the exponentials shows it, and propagates without; ba, r, val: this lane's part of the argmax, the sums
// and the value row, to be joined with the other lane's.
struct TileOut {
  float best;
  int32_t ba;
  RlSums r;
  float val;
};
template <int AT>
__device__ __forceinline__ TileOut tile_out(KernArgs a, bool rl, uint64_t am, uint32_t id, int32_t e,
                                            const f32x16 (&acc)[AT], int g) {
  TileOut o;
  const MaskWords m = mask_words(am, g);
  constexpr int AA = action_tiles(AT);
  const uint32_t low = rl ? ~0u : minus_inf();   // what a masked logit becomes: NaN where NaN is passed over (one v_or_b32)
  float zm[AA][16];
  float best = __uint_as_float(low);
#pragma unroll
  for (int T = 0; T < AA; ++T)
#pragma unroll
    for (int v = 0; v < 16; ++v) zm[T][v] = mask_logit(acc[T][v], bit_ones(m.w[T], 8 * (v >> 2) + (v & 3)), low);
  int32_t x, y;
  if (rl) {   // uniform
#pragma unroll
    for (int T = 0; T < AA; ++T)
#pragma unroll
      for (int v = 0; v < 16; v += 2) best = max3(best, zm[T][v], zm[T][v + 1]);
    swap_halves<32>(as_int(best), x, y);
    best = max3(__int_as_float(x), __int_as_float(y), __int_as_float(y));
  } else {
#pragma unroll
    for (int T = 0; T < AA; ++T)
#pragma unroll
      for (int v = 0; v < 16; v += 2) best = maximum3(best, zm[T][v], zm[T][v + 1]);
    swap_halves<32>(as_int(best), x, y);
    best = maximum3(__int_as_float(x), __int_as_float(y), __int_as_float(y));
  }
  o.best = best;
  o.ba = 127;
  if (!rl || a->greedy) {   // uniform
    int32_t ba = 127;
#pragma unroll
    for (int T = AA - 1; T >= 0; --T)
#pragma unroll
      for (int v = 15; v >= 0; --v) ba = zm[T][v] == best ? 32 * T + 8 * (v >> 2) + (v & 3) : ba;
    o.ba = ba + 4 * g;
  }
  o.val = 0.f;
  if (!rl) return o;
  const bool sample = a->greedy == 0;
  // the key schedule is formed per row group: hoisted out of the kernel's loop
  // its 18 words would spill scalar registers into vector ones
  uint32_t k0 = a->seed_lo, k1 = a->seed_hi;
  asm volatile("" : "+s"(k0), "+s"(k1));
#pragma unroll
  for (int T = 0; T < AT; ++T) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int a0 = 32 * T + 8 * j;   // the lane pair's 8 actions: two Philox blocks
      const float z[4] = {acc[T][4 * j], acc[T][4 * j + 1], acc[T][4 * j + 2], acc[T][4 * j + 3]};
      if (T < AA && a0 < a->A) {        // uniform
        const uint32_t mb = m.w[T < AA ? T : 0] >> (8 * j);
        if (sample) {
          const uint4 w = philox10(make_uint4(id, (uint32_t)e, (uint32_t)((a0 >> 2) + g), 0u), k0, k1);
          rl_block<true>(o.r, z, mb, best, a0 + 4 * g, w);
        } else {
          rl_block<false>(o.r, z, mb, best, a0 + 4 * g, make_uint4(0, 0, 0, 0));
        }
      }
      if (a->value && (a->A >> 3) == 4 * T + j) {   // uniform: the group of row A
        const int i = a->A & 3;
        const float v = i == 0 ? z[0] : (i == 1 ? z[1] : (i == 2 ? z[2] : z[3]));
        o.val = ((a->A >> 2) & 1) == g ? v : 0.f;
      }
    }
  }
  return o;
}

// A tile's logits, 32 rows from row r0 on (the row's other lane stores the rest).
template <int AT>
__device__ __forceinline__ void store_tile_logits(KernArgs a, int32_t r, int32_t bad, const f32x16 (&acc)[AT], int g) {
  float* out = a->logits + (size_t)r * a->A;
#pragma unroll
  for (int T = 0; T < AT; ++T) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float z0 = bad ? 0.f : acc[T][4 * j], z1 = bad ? 0.f : acc[T][4 * j + 1];
      const float z2 = bad ? 0.f : acc[T][4 * j + 2], z3 = bad ? 0.f : acc[T][4 * j + 3];
      store_logits(a, out, 32 * T + 8 * j + 4 * g, z0, z1, z2, z3);
    }
  }
}

// The action of a row from its joined argmax and its largest logit: -1 when no
// action is valid, the first valid one when none exceeds -inf, which masked
// actions equal too (or when no logit is left beside NaN).
__device__ __forceinline__ int32_t argmax_of(int32_t ba, uint64_t am, float best) {
  return ba >= 64 || best == __uint_as_float(kMinusInf) ? __ffsll((unsigned long long)am) - 1 : ba;
}
// The action of a row with a NaN among its valid logits; with RL outputs (no
// ARGMAX) only where its first valid one is NaN, which then is drawn too.
template <bool ARGMAX>
__device__ __forceinline__ void scan_store(KernArgs a, const RowCtx& c, const NanScan& f) {
  if (!c.bad && (ARGMAX || f.first_nan)) a->actions[c.r] = argmax_of(f.first_nan ? 127 : f.ba, c.amask, f.best);
}

// Masked argmax over the lane pair (n, n + 32), logits store, action store (or
// the RL-rollout outputs). RL: 0 = greedy route only, 1 = RL outputs only, 2 =
// either, chosen by a.rl at run time.
template <int AT, int RL = 2>
__device__ __forceinline__ void epilogue(const RowCtx& c, const f32x16 (&acc)[AT], int g) {
  const KernArgs a = late_args();
  const bool rl = RL == 1 || (RL == 2 && a->rl);
  uint64_t am = c.amask;
  asm volatile("" : "+v"(am));   // the shifted mask is formed here, not kept beside the mask since the row's setup
  uint32_t id = 0;
  if (rl && a->greedy == 0) id = c.id >= 0 ? (uint32_t)c.id : request_id(a, c);
  TileOut o = tile_out<AT>(a, rl, am, id, c.e, acc, g);
  int32_t x, y;
  swap_halves<32>(o.ba, x, y);
  const int32_t ba = argmax_of(x < y ? x : y, c.amask, o.best);
  if (rl) {
    auto other = [](float v) { return __int_as_float(xshfl<32>(as_int(v))); };
    rl_join(o.r, other(o.r.s), other(o.r.sz), other(o.r.bs), other(o.r.bz), xshfl<32>(o.r.ba));
    o.val += other(o.val);   // one lane of the pair holds row A
  }
  if (c.live && g == 0) {
    if (rl) {
      rl_store(a, c, o.r, o.best, ba, o.val);
    } else {
      a->actions[c.r] = c.bad ? -1 : ba;
      if (c.bad) atomicOr(a->err, c.bad);
    }
  }
  if (c.live && a->logits) store_tile_logits<AT>(a, c.r, c.bad, acc, g);
  const float sign = rl ? o.r.s : o.best;
  if (ballot(sign != sign) != 0) {
    const NanScan f = nan_scan<AT, RL != 1>(c.amask, acc, g);
    if (sign != sign && c.live && g == 0) {
      if (rl) scan_store<false>(a, c, f);
      else scan_store<true>(a, c, f);
    }
  }
}

// Two registers v0, v1 that hold tile 0's and tile 1's value in every lane pair:
// x gets the lower lane's and y the upper lane's value of the row this lane owns
// (lane l: row l of the 64, the lower half of the lanes tile 0's rows).
__device__ __forceinline__ void own_halves(int32_t v0, int32_t v1, int32_t& x, int32_t& y) {
  const auto r = __builtin_amdgcn_permlane32_swap(v0, v1, false, false);
  x = (int32_t)r[0];
  y = (int32_t)r[1];
}
// This lane's value of the row it owns, handed to both lanes of the tiles' pairs:
// t[0] for tile 0's row, t[1] for tile 1's.
__device__ __forceinline__ void spread(int32_t v, int32_t (&t)[2]) { swap_halves<32>(v, t[0], t[1]); }

// The same outputs for a wave tile of 64 rows (two 32-row MFMA tiles) whose row
// contexts lie one per lane: c is lane l's row r0 + l. The parts of a row meet in
// the lane that owns it, so what follows the matrix work per row (softmax
// normalisation, stores) runs once per 64 rows on full lanes.
template <int AT, int RL>
__device__ __forceinline__ void epilogue64(const RowCtx& c, const f32x16 (&acc)[2][AT], int g) {
  static_assert(RL == 0 || RL == 1, "greedy or RL outputs");
  const KernArgs a = late_args();
  uint64_t am = c.amask;
  asm volatile("" : "+v"(am));
  int32_t lo[2], hi[2], id[2] = {0, 0}, e[2] = {0, 0};
  spread((int32_t)(uint32_t)am, lo);
  spread((int32_t)(am >> 32), hi);
  if (RL && a->greedy == 0) {
    spread((int32_t)request_id(a, c), id);
    spread(c.e, e);
  }
  TileOut o[2];
#pragma unroll
  for (int j = 0; j < 2; ++j)
    o[j] = tile_out<AT>(a, RL == 1, (uint64_t)(uint32_t)hi[j] << 32 | (uint32_t)lo[j], (uint32_t)id[j], e[j], acc[j], g);
  int32_t x, y;
  own_halves(o[0].ba, o[1].ba, x, y);
  const float best = g ? o[1].best : o[0].best;
  const int32_t ba = argmax_of(x < y ? x : y, am, best);
  RlSums r;
  float val = 0.f;
  if constexpr (RL == 1) {
    auto meet = [](float v0, float v1, float& p, float& q) {
      int32_t s, t;
      own_halves(as_int(v0), as_int(v1), s, t);
      p = __int_as_float(s);
      q = __int_as_float(t);
    };
    float s, sz, bs, bz, v0, v1;
    meet(o[0].r.s, o[1].r.s, r.s, s);
    meet(o[0].r.sz, o[1].r.sz, r.sz, sz);
    meet(o[0].r.bs, o[1].r.bs, r.bs, bs);
    meet(o[0].r.bz, o[1].r.bz, r.bz, bz);
    own_halves(o[0].r.ba, o[1].r.ba, r.ba, x);
    rl_join(r, s, sz, bs, bz, x);
    meet(o[0].val, o[1].val, v0, v1);   // one lane of the pair holds row A
    val = v0 + v1;
  }
  if (c.live) {
    if constexpr (RL == 1) {
      rl_store(a, c, r, best, ba, val);
    } else {
      a->actions[c.r] = c.bad ? -1 : ba;
      if (c.bad) atomicOr(a->err, c.bad);
    }
  }
  if (a->logits) {
    int32_t bad[2], row[2];
    spread(c.bad, bad);
    spread(c.live ? c.r : -1, row);
#pragma unroll
    for (int j = 0; j < 2; ++j)
      if (row[j] >= 0) store_tile_logits<AT>(a, row[j], bad[j], acc[j], g);
  }
  const float sign = RL == 1 ? r.s : best;
  if (ballot(sign != sign) != 0) {
    // the scan of both tiles, for the row this lane owns
    uint64_t m = c.amask;
    asm volatile("" : "+v"(m));
    spread((int32_t)(uint32_t)m, lo);
    spread((int32_t)(m >> 32), hi);
    const NanScan f0 = nan_scan<AT, RL == 0>((uint64_t)(uint32_t)hi[0] << 32 | (uint32_t)lo[0], acc[0], g);
    const NanScan f1 = nan_scan<AT, RL == 0>((uint64_t)(uint32_t)hi[1] << 32 | (uint32_t)lo[1], acc[1], g);
    if (sign != sign && c.live) scan_store<RL == 0>(a, c, g ? f1 : f0);
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

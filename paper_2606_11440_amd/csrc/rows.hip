// Rows of a tick in a pool with multi-step agent chains (Sec. 4.3).
//
// An env's rows at tick t are its pending calls (spawned by completions at
// t - 1, in spawn order), then its arrivals in arrival order. The route step
// evaluates the policy on the flat row space; these kernels build it: one
// block scans the per-env row counts into row offsets, then one wave per env
// writes each row's query-embedding row, remaining budget and role.
#include "im_internal.h"
#include "wave.h"

namespace im {
namespace {

constexpr int kScanThreads = 1024;

// Arrivals of env e the route step takes: a CSR entry outside the arrays
// contributes none (the schedule step reports it and skips the env).
__device__ __forceinline__ int32_t usable(const RowsArgs& a, int32_t lo, int32_t hi) {
  return (lo < 0 || hi < lo || hi > a.n_total || hi - lo > a.max_arrivals) ? 0 : hi - lo;
}

// One block: exclusive scan of (pending + usable arrivals) over the envs.
// Each thread holds the counts of kPer consecutive envs in registers; wave
// scans by shuffles, the 16 wave totals scanned by the first wave; blocks of
// 1024 * kPer envs in sequence with a carried total. Latency-bound: the tick,
// the offsets and the pending counts of both parities (the tick picks one) are
// in flight together, and the CSR is checked on the offsets already loaded.
// 4,096 envs: 8.1 -> 6.4 us (three dependent round trips before). The next block's
// loads travel during a block's scan: 65,536 envs 82.4 -> 71.1 us (79.3 with 8 envs
// per thread and no load ahead).
constexpr int kPer = 4;

__device__ __forceinline__ int32_t wave_incl_scan(int32_t x, int lane) {
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int32_t y = __shfl_up(x, d, 64);
    if (lane >= d) x += y;
  }
  return x;
}

// MANY: more envs than one pass takes (4,096 envs without the loop: 6.2 -> 5.7 us).
template <bool MANY>
__global__ __launch_bounds__(kScanThreads) void rows_scan_kernel(RowsArgs a) {
  constexpr int NWAVE = kScanThreads / 64;
  __shared__ int32_t wsum[NWAVE];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  // envs tid kPer + j of the block of envs at base: their offsets and the
  // pending counts of either parity
  int32_t off[kPer + 1], pc0[kPer], pc1[kPer];
  auto load = [&](int base) {
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
      const int e = min(base + tid * kPer + j, a.E - 1);
      off[j] = a.offsets[min(base + tid * kPer + j, a.E)];
      pc0[j] = a.pcnt[e];
      pc1[j] = a.pcnt[(size_t)a.E + e];
    }
    off[kPer] = a.offsets[min(base + tid * kPer + kPer, a.E)];
  };
  load(0);
  const int32_t t = a.ms[0].t;
  const int32_t first = a.offsets[0], total = a.offsets[a.E];
  // The rows are laid out by a scan over the arrival CSR, so it must be one
  // monotone partition of [0, n_total); otherwise no arrival is usable (every
  // env then skips the tick in the schedule step).
  int broken = first != 0 || total != a.n_total;
#pragma unroll
  for (int j = 0; j < kPer; ++j) broken |= tid * kPer + j < a.E && off[j + 1] < off[j];
  for (int e = kScanThreads * kPer + tid; MANY && e < a.E; e += kScanThreads) broken |= a.offsets[e + 1] < a.offsets[e];
  const bool whole = __syncthreads_or(broken) == 0;
  int32_t carry = 0;
  for (int base = 0; base < a.E; base += kScanThreads * kPer) {
    int32_t c[kPer];
    int32_t sum = 0;
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
      const int e = base + tid * kPer + j;
      c[j] = e < a.E ? ((t & 1) ? pc1[j] : pc0[j]) + (whole ? usable(a, off[j], off[j + 1]) : 0) : 0;
      sum += c[j];
    }
    if (MANY && base + kScanThreads * kPer < a.E) load(base + kScanThreads * kPer);   // in flight during this block's scan
    const int32_t x = wave_incl_scan(sum, lane);
    if (lane == 63) wsum[w] = x;
    __syncthreads();
    if (w == 0) {
      const int32_t v = wave_incl_scan(lane < NWAVE ? wsum[lane] : 0, lane);
      if (lane < NWAVE) wsum[lane] = v;
    }
    __syncthreads();
    int32_t run = carry + (w > 0 ? wsum[w - 1] : 0) + x - sum;
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
      const int e = base + tid * kPer + j;
      if (e < a.E) a.roff[e] = run;
      run += c[j];
    }
    carry += wsum[NWAVE - 1];
    if (!MANY) break;
    __syncthreads();   // wsum is rewritten by the next block of envs
  }
  if (tid == 0) {
    a.roff[a.E] = carry;
    a.n_rows[0] = carry;
    a.n_rows[1] = whole ? 0 : 1;
  }
}

// One wave per env: the pending calls' rows (query row, deadline - t, role of
// call k: (role0 + k) mod n_roles), then the arrivals' rows.
__global__ __launch_bounds__(256) void rows_gather_kernel(RowsArgs a) {
  const int lane = threadIdx.x & 63;
  const int e = (int)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (e >= a.E) return;
  const int32_t t = a.ms[0].t;
  const int32_t pc0 = a.pcnt[e], pc1 = a.pcnt[(size_t)a.E + e];   // both parities, not waiting for the tick
  const int32_t lo = a.offsets[e], hi = a.offsets[e + 1], whole = a.n_rows[1] == 0;   // n_rows: the scan kernel's
  const int32_t base = a.roff[e];
  const int32_t pc = (t & 1) ? pc1 : pc0;
  const int4* pend = a.pend + ((size_t)(t & 1) * a.E + e) * a.pend_cap;
  const int32_t na = whole ? usable(a, lo, hi) : 0;
  for (int i = lane; i < pc; i += 64) {
    const int4 p = pend[i];
    a.rq[base + i] = chain_q(p.x);
    a.rb[base + i] = (int16_t)remaining_budget(p.z, t);
    a.rr[base + i] = (int16_t)(a.n_roles > 0 ? (chain_role0(p.y) + chain_k(p.x)) % a.n_roles : 0);
  }
  for (int i = lane; i < na; i += 64) {
    a.rq[base + pc + i] = a.q_idx[lo + i];
    a.rb[base + pc + i] = a.budget[lo + i];
    a.rr[base + pc + i] = a.role ? a.role[lo + i] : (int16_t)0;
  }
}

}  // namespace

hipError_t launch_rows(const RowsArgs& a, hipStream_t s) {
  if (a.E > kScanThreads * kPer) hipLaunchKernelGGL(rows_scan_kernel<true>, dim3(1), dim3(kScanThreads), 0, s, a);
  else hipLaunchKernelGGL(rows_scan_kernel<false>, dim3(1), dim3(kScanThreads), 0, s, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(rows_gather_kernel, dim3((unsigned)((a.E + 3) / 4)), dim3(256), 0, s, a);
  return hipGetLastError();
}

}  // namespace im

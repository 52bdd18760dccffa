// Radix-2 forward procedure for K = 8 and 9: dispatch, the kernel for int8 soft
// values of rate 1/4 codes and its check of frames split in time.  The packed
// int8 kernel (beta <= 3) is in mivit_fwd_wpk.hip, the float kernels in
// mivit_fwd_wide_f32.hip and mivit_fwd_wide_f16.hip.
#include "mivit_fwd_wide.h"

namespace mivit {

namespace wide {

// Branch metrics are read from LDS kPrefetch stages ahead of their use: a
// lone wavefront (the longest frame of a batch, once the others are done)
// otherwise waits out the LDS latency at every stage.
constexpr int kPrefetch = 3;

template <int KM1, int DT, int R, int NP, int P0, int K>
__device__ __forceinline__ void fetch_bm(typename Ty<DT>::T (&dst)[R],
                                         const typename Ty<DT>::T* bmt,
                                         const int (&pat)[KM1][R]) {
  constexpr int Q = (P0 + K) % KM1;
#pragma unroll
  for (int r = 0; r < R; ++r) dst[r] = bmt[K * NP + pat[Q][r]];
}

// Stages K0..31 of a full block starting at phase P0 (static phases); q
// holds the branch metrics of stages K0 .. K0 + kPrefetch - 1.
template <int KM1, int DT, int R, int NP, int P0, int K0>
__device__ __forceinline__ void stages_full(Wave<DT, R>& W, const typename Ty<DT>::T* bmt,
                                            const int (&pat)[KM1][R],
                                            typename Ty<DT>::T (&q)[kPrefetch][R]) {
  if constexpr (K0 < 32) {
    constexpr int Q = (P0 + K0) % KM1;
    typename Ty<DT>::T bm[R];
#pragma unroll
    for (int r = 0; r < R; ++r) bm[r] = q[K0 % kPrefetch][r];
    if constexpr (K0 + kPrefetch < 32)
      fetch_bm<KM1, DT, R, NP, P0, K0 + kPrefetch>(q[K0 % kPrefetch], bmt, pat);
    stage<KM1, DT, R, Q>(W, bm);
    __builtin_amdgcn_sched_barrier(0);  // keep the reads ahead of their stages
    stages_full<KM1, DT, R, NP, P0, K0 + 1>(W, bmt, pat, q);
  }
}

template <int KM1, int DT, int R, int NP, int P0, int K>
__device__ __forceinline__ void prefetch_first(typename Ty<DT>::T (&q)[kPrefetch][R],
                                               const typename Ty<DT>::T* bmt,
                                               const int (&pat)[KM1][R]) {
  if constexpr (K < kPrefetch) {
    fetch_bm<KM1, DT, R, NP, P0, K>(q[K], bmt, pat);
    prefetch_first<KM1, DT, R, NP, P0, K + 1>(q, bmt, pat);
  }
}

struct Ctx {
  int64_t offset;  // integer metrics: total subtracted by renormalisation
  int S, lane;     // S: one past the last stage this unit runs
  int t_store;     // first stage whose decisions are stored
  int32_t* v_start;  // split part after the first: boundary record to fill at t_store
  int64_t* m_start;
  uint8_t* pend_dst;  // where the pending decision words go, or null
};

// One block of up to 32 stages starting at tb; BI its index in the period
// of the phase pattern.  lv: this lane's soft values of stage tb + lane
// (lanes < 32), replaced by those of the next block.
template <int KM1, int DT, int BETA, int BI, int R>
__device__ __forceinline__ void one_block(Wave<DT, R>& W, Ctx& cx, typename Ty<DT>::T* bmt,
                                          const typename Ty<DT>::In* llr,
                                          typename Ty<DT>::T (&lv)[BETA],
                                          const int (&pat)[KM1][R], uint64_t* sv, int tb) {
  using T = typename Ty<DT>::T;
  constexpr int NP = 1 << BETA;
  const int n = min(32, cx.S - tb);
  if (cx.lane < 32) {
#pragma unroll
    for (int p = 0; p < NP / 2; ++p) {
      T v = (T)0;
#pragma unroll
      for (int b = 0; b < BETA; ++b) v += ((p >> b) & 1) ? -lv[b] : lv[b];
      bmt[cx.lane * NP + p] = v;
      bmt[cx.lane * NP + (NP - 1 - p)] = -v;
    }
  }
  {
    const int t = tb + 32 + cx.lane;
    const bool ok = cx.lane < 32 && t < cx.S;
#pragma unroll
    for (int b = 0; b < BETA; ++b) lv[b] = ok ? (T)llr[(int64_t)t * BETA + b] : (T)0;
  }
  // the previous block's decisions go out here, after the next soft values
  // are requested: the memory counter the next block start waits on (for
  // those soft values) covers stores too, so stores issued at the end of a
  // block would hold up the start of the next
  if (cx.pend_dst) store_block<KM1, R>(cx.pend_dst, W.pend);
  if constexpr (Ty<DT>::kInt) {
    if (tb > 0) {
      // renormalise by the metric of state 0 (always position 0: lane 0, register 0)
      const T ref = __builtin_amdgcn_readfirstlane(W.pm[0]);
#pragma unroll
      for (int r = 0; r < R; ++r) W.pm[r] -= ref;
      cx.offset += ref;
    }
    if (cx.v_start && tb == cx.t_store) {
      // a later part of a split frame, at the end of its warm-up
#pragma unroll
      for (int r = 0; r < R; ++r) cx.v_start[64 * r + cx.lane] = (int32_t)W.pm[r];
      if (cx.lane == 0) *cx.m_start = cx.offset;
    }
  }
  wave_sync();
  constexpr int P0 = (32 * BI) % KM1;
  if (n == 32) {
    T q[kPrefetch][R];
    prefetch_first<KM1, DT, R, NP, P0, 0>(q, bmt, pat);
    stages_full<KM1, DT, R, NP, P0, 0>(W, bmt, pat, q);
  } else {
#pragma unroll 1
    for (int k = 0; k < n; ++k) stage_dyn<KM1, DT, R, NP, 0>(W, bmt + k * NP, pat, (P0 + k) % KM1);
  }
  // this block's decisions: stored at the next block's start, or after the
  // last block
  cx.pend_dst = nullptr;
  if (tb >= cx.t_store) {
    cx.pend_dst = (uint8_t*)sv + (int64_t)(tb >> 3) * (1 << KM1) + cx.lane;
#pragma unroll
    for (int r = 0; r < R; ++r) W.pend[r] = n == 32 ? W.acc[r] : W.acc[r] << (32 - n);
  }
#pragma unroll
  for (int r = 0; r < R; ++r) W.acc[r] = 0;
  wave_sync();
}

template <int KM1, int DT, int BETA, int BI, int NB, int R>
__device__ __forceinline__ void super_block(Wave<DT, R>& W, Ctx& cx, typename Ty<DT>::T* bmt,
                                            const typename Ty<DT>::In* llr,
                                            typename Ty<DT>::T (&lv)[BETA],
                                            const int (&pat)[KM1][R], uint64_t* sv, int t0) {
  if constexpr (BI < NB) {
    const int tb = t0 + 32 * BI;
    if (tb < cx.S) {
      one_block<KM1, DT, BETA, BI, R>(W, cx, bmt, llr, lv, pat, sv, tb);
      super_block<KM1, DT, BETA, BI + 1, NB, R>(W, cx, bmt, llr, lv, pat, sv, t0);
    }
  }
}

}  // namespace wide

// One wavefront per unit: a whole item (frame or chunk window), or one part
// of a frame split in time (kind 0), or a repair
// of one (kind 1, unit count read from the device).  A part after the first
// runs `warm` stages from all-zero metrics before it_begin and keeps no
// decisions from them; a part before the last leaves its end metrics in a
// boundary record, the last part its own metric, which the check completes.
template <int KM1, int BETA>
__global__ __launch_bounds__(64 * wide::kWideWaves, 4) void k_fwd_wide(
    const DevCode* __restrict__ codes, const Item* __restrict__ items,
    const SplitUnit* __restrict__ units, int n_units, const int32_t* dev_count, int kind,
    WideBound* bounds, int64_t* last_m, const int64_t* rep_m0,
    const int8_t* __restrict__ llr_all, uint64_t* __restrict__ surv, int64_t* metric,
    int32_t* end_out, int32_t* item_end) {
  using namespace wide;
  constexpr int DT = 1;
  using T = int;
  constexpr int R = 1 << (KM1 - 6), NS = 1 << KM1, NP = 1 << BETA;
  constexpr int SUPER = 32 * KM1 / gcd_c(32, KM1);  // lcm(32, K-1)
  __shared__ T bmt_all[kWideWaves][32 * NP];
  __shared__ T xpm_all[kWideWaves][NS];
  const int wid = threadIdx.x >> 6;
  const int lane = threadIdx.x & 63;
  if (dev_count) n_units = min(n_units, __builtin_amdgcn_readfirstlane(*dev_count));
  // (uniform, so that the unit, item and code stay out of the vector registers:
  // with them K = 9 fitted three wavefronts to a SIMD where plans cut batches for
  // four, and 4096 frames of 8192 bits took 1891 us instead of 1568)
  const int u = __builtin_amdgcn_readfirstlane(blockIdx.x * kWideWaves + wid);
  if (u >= n_units) return;  // no workgroup barriers: safe to leave
  const SplitUnit U = units[u];
  const Item it = items[U.first];
  const DevCode c = codes[it.code];
  const int8_t* llr = llr_all + it.llr_off;
  uint64_t* sv = surv + it.surv_off;
  T* bmt = bmt_all[wid];
  T* xpm = xpm_all[wid];
  const bool first_part = kind == 0 && U.part == 0;
  const bool split = U.n_parts > 1;
  const int s0 = U.it_begin - U.warm;  // a multiple of SUPER: phases start at 0

  // table offset (pattern) of position 64 r + lane at each phase: the even
  // previous state's branch into the state held there after the stage
  int pat[KM1][R];
  patterns<KM1, DT, R>(pat, c, lane, 0);
  Wave<DT, R> W;
  W.xch = nullptr;
  W.nw = 1;
  W.fw = 0;
  W.xb = 0;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    if (first_part)
      W.pm[r] = (it.start_known && (r != 0 || lane != 0)) ? Ty<DT>::unreachable() : (T)0;
    else if (kind == 0)
      W.pm[r] = (T)0;  // a later part: all-zero metrics (unknown start)
    else
      W.pm[r] = Ty<DT>::from(bounds[U.bnd + U.part - 1].v_end[64 * r + lane]);  // repair
    W.acc[r] = 0;
  }
  Ctx cx{0, U.it_end, lane, U.it_begin, nullptr, nullptr, nullptr};
  if (kind == 0 && U.part > 0) {
    cx.v_start = bounds[U.bnd + U.part - 1].v_start;
    cx.m_start = &bounds[U.bnd + U.part - 1].m_start;
  }
  T lv[BETA];
  {
    const bool ok = lane < 32 && s0 + lane < cx.S;
#pragma unroll
    for (int b = 0; b < BETA; ++b) lv[b] = ok ? (T)llr[(int64_t)(s0 + lane) * BETA + b] : (T)0;
  }
  for (int t0 = s0; t0 < cx.S; t0 += SUPER)
    super_block<KM1, DT, BETA, 0, SUPER / 32, R>(W, cx, bmt, llr, lv, pat, sv, t0);
  if (cx.pend_dst) store_block<KM1, R>(cx.pend_dst, W.pend);

  {
    if (kind == 0 && split && U.part < U.n_parts - 1) {
      // the end of a part before the last: range control as at a block
      // start, then the boundary record
      const T ref = __builtin_amdgcn_readfirstlane(W.pm[0]);
      WideBound& B = bounds[U.bnd + U.part];
#pragma unroll
      for (int r = 0; r < R; ++r) B.v_end[64 * r + lane] = (int32_t)(W.pm[r] - ref);
      if (lane == 0) B.m_end = cx.offset + ref;
      return;
    }
  }

  const int S = cx.S;
  int js;
  const T vj = end_state<KM1, DT, R, 1>(W.pm, S, lane, 0, it.end_state, xpm, nullptr, nullptr, js);
  if (lane == 0) {
    item_end[it.slot] = js;
    if (it.frame >= 0 && end_out) end_out[it.frame] = js;
    const int64_t local = (int64_t)vj + cx.offset;
    if (kind == 0 && split)
      last_m[it.slot] = local;  // completed by the check
    else if (it.frame >= 0 && metric)
      metric[it.frame] = local + (kind == 1 ? rep_m0[it.slot] : 0);
  }
}

// The check after a split forward pass of the K = 8, 9 kernel, one wavefront
// per split frame (its part-0 unit): boundary k is exact when part k's
// range-controlled metrics at its end equal part k+1's after its warm-up at
// every position; then the metric is the last part's plus the accumulated
// constants, else a repair unit restarts the frame at the first inexact
// boundary from the true metrics.
__global__ __launch_bounds__(64 * wide::kWideWaves) void k_wide_check(
    const DevCode* __restrict__ codes, const Item* __restrict__ items,
    const SplitUnit* __restrict__ split, int n_split, const SplitUnit* __restrict__ units,
    const WideBound* __restrict__ bounds, const int64_t* __restrict__ last_m, int64_t* rep_m0,
    SplitUnit* rep_units, int32_t* rep_count, int64_t* metric) {
  const int lane = threadIdx.x & 63;
  const int e = blockIdx.x * wide::kWideWaves + (threadIdx.x >> 6);
  if (e >= n_split) return;
  const SplitUnit U = split[e];
  const Item it = items[U.first];
  const int NS = 1 << (codes[it.code].K - 1);  // positions compared
  const int n_b = U.n_parts - 1;
  int64_t T = bounds[U.bnd].m_end;  // part 0 is exact
  int64_t D = 0;
  int fail = -1;
  for (int b = 0; b < n_b; ++b) {
    const WideBound& B = bounds[U.bnd + b];
    bool diff = false;
    for (int p = lane; p < NS; p += 64) diff = diff || (B.v_end[p] != B.v_start[p]);
    if (__ballot(diff) != 0) {
      fail = b;
      break;
    }
    D = T - B.m_start;
    if (b + 1 < n_b) T = bounds[U.bnd + b + 1].m_end + D;
  }
  if (lane != 0) return;
  if (fail < 0) {
    if (metric && it.frame >= 0) metric[it.frame] = last_m[it.slot] + D;
    return;
  }
  rep_m0[it.slot] = T;
  SplitUnit R = U;
  R.it_begin = units[U.warm + fail + 1].it_begin;
  R.it_end = it.n_stages;
  R.warm = 0;
  R.part = fail + 1;
  rep_units[atomicAdd(rep_count, 1)] = R;
}

hipError_t launch_zero_i32(int32_t* p, int n, hipStream_t st);
hipError_t launch_fwd_wpk(int K, int beta, const DevCode* codes, const Item* items,
                          const SplitUnit* units, int n_units, const int8_t* llr, uint64_t* surv,
                          int64_t* metric, int32_t* end_out, int32_t* item_end, WideBound* bounds,
                          int64_t* last_m, const SplitUnit* split, int n_split, int64_t* rep_m0,
                          hipStream_t st);
hipError_t launch_wide_f32(int K, int beta, int wpf, const DevCode* codes, const Item* items,
                           const SplitUnit* units, int n_units, const void* llr, uint64_t* surv,
                           void* metric, int32_t* end_out, int32_t* item_end, hipStream_t st);
hipError_t launch_wide_f16(int K, int beta, int wpf, const DevCode* codes, const Item* items,
                           const SplitUnit* units, int n_units, const void* llr, uint64_t* surv,
                           void* metric, int32_t* end_out, int32_t* item_end, hipStream_t st);

hipError_t launch_fwd_wide(int K, int beta, int dt, int wpf, bool packed, const DevCode* codes,
                           const Item* items,
                           const SplitUnit* units, int n_units, const void* llr, uint64_t* surv,
                           void* metric, int32_t* end_out, int32_t* item_end, WideBound* bounds,
                           int64_t* last_m, const SplitUnit* split, int n_split, int64_t* rep_m0,
                           SplitUnit* rep_units, int32_t* rep_count, hipStream_t st) {
  if (n_units <= 0) return hipSuccess;
  if (n_split > 0 && dt != 1) return hipErrorInvalidValue;  // split frames: int8 only
  if (wpf != 1 && ((wpf != 2 && !(wpf == 4 && K == 9)) || dt == 1)) return hipErrorInvalidValue;
  if (packed && (dt != 1 || wpf != 1 || beta > 3)) return hipErrorInvalidValue;
  if (dt != 1) {
    return dt == 0   ? launch_wide_f32(K, beta, wpf, codes, items, units, n_units, llr, surv,
                                       metric, end_out, item_end, st)
           : dt == 2 ? launch_wide_f16(K, beta, wpf, codes, items, units, n_units, llr, surv,
                                       metric, end_out, item_end, st)
                     : hipErrorInvalidValue;
  }
  if (packed)
    return launch_fwd_wpk(K, beta, codes, items, units, n_units, (const int8_t*)llr, surv,
                          (int64_t*)metric, end_out, item_end, bounds, last_m, split, n_split,
                          rep_m0, st);
  const dim3 block(64 * wide::kWideWaves);
  const dim3 grid((n_units + wide::kWideWaves - 1) / wide::kWideWaves);
  const dim3 grid_rep((n_split + wide::kWideWaves - 1) / wide::kWideWaves);
  hipError_t e = hipSuccess;
#define MV_WIDE(KM1)                                                                             \
  do {                                                                                           \
    hipLaunchKernelGGL((k_fwd_wide<KM1, 4>), grid, block, 0, st, codes, items, units, n_units,   \
                       (const int32_t*)nullptr, 0, bounds, last_m, (const int64_t*)nullptr,      \
                       (const int8_t*)llr, surv, (int64_t*)metric, end_out, item_end);           \
    e = hipGetLastError();                                                                        \
    if (e != hipSuccess || n_split <= 0) return e;                                                \
    e = launch_zero_i32(rep_count, 1, st);                                                        \
    if (e != hipSuccess) return e;                                                                \
    hipLaunchKernelGGL(k_wide_check, grid_rep, block, 0, st, codes, items, split, n_split,        \
                       units, (const WideBound*)bounds, (const int64_t*)last_m, rep_m0,           \
                       rep_units, rep_count, (int64_t*)metric);                                   \
    e = hipGetLastError();                                                                        \
    if (e != hipSuccess) return e;                                                                \
    hipLaunchKernelGGL((k_fwd_wide<KM1, 4>), grid_rep, block, 0, st, codes, items,               \
                       (const SplitUnit*)rep_units, n_split, (const int32_t*)rep_count, 1, bounds,\
                       last_m, (const int64_t*)rep_m0, (const int8_t*)llr, surv,                  \
                       (int64_t*)metric, end_out, item_end);                                      \
    return hipGetLastError();                                                                     \
  } while (0)
  // the 32-bit kernel serves the codes whose metrics do not fit 16 bits
  switch (K * 8 + beta) {
    case 8 * 8 + 4: MV_WIDE(7);
    case 9 * 8 + 4: MV_WIDE(8);
    default: return hipErrorInvalidValue;
  }
#undef MV_WIDE
}

}  // namespace mivit

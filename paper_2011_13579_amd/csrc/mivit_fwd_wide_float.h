// Radix-2 forward procedure for K = 8 and 9, float32 and float16 soft values:
// WPF wavefronts per frame (1, 2 or 4), R = 2^(K-1)/(64 WPF) states per lane.
//
// The state map is that of mivit_fwd_wide.h.  A stage takes the maximum of
// the candidates and shifts the sign bit of their difference into the
// position's decision word, as in the K <= 7 kernel (mivit_fwd_rot.h), whose
// exchanges, conditions on the soft values and loop for the others apply
// here too.
//
// What bounds it.  One frame alone is a latency chain per stage; a full
// device is bound by vector instructions: 5 to 7 per state (by phase) and
// stage, 5.9 on average for K = 9.  So that nothing else enters the chain,
// branch metrics are read from LDS P stages ahead, the table they come from
// is written 16 stages (a half block) ahead into the half last read, and
// the soft values are loaded NR half blocks ahead.  The two new states of a
// butterfly between registers share one branch metric with opposite signs.
//
// Forward pass, K = 9 rate 1/3, against one compare, select and mask per state
// and stage: one frame of 4096 bits 365 -> 235 us on one wavefront, 233 -> 175
// on four; 1024 frames 387 -> 257 on one; 4096 of 2000 bits 361 -> 344.
//
// Several wavefronts per frame: the stages whose phase is a wavefront bit
// exchange the metrics through LDS with one barrier; the others run on 1/WPF
// of the registers.
#pragma once
#include <utility>

#include "mivit_fwd_rot.h"
#include "mivit_fwd_wide.h"

namespace mivit {

namespace wide {

// A wavefront's table: 32 rows of 2^BETA patterns, stored by 16 bytes (rate 1/2:
// by words, as the compiler combines them best).
template <int BETA>
struct alignas(BETA == 2 ? alignof(float) : 16) WfTable {
  float w[32 << BETA];
};

template <int KM1, int DT, int BETA, int WPF>
struct Wf {
  using In = typename Ty<DT>::In;
  static constexpr int NS = 1 << KM1, NP = 1 << BETA;
  static constexpr int R = (1 << (KM1 - 6)) / WPF;
  static constexpr int P = R >= 4 ? 4 : 8;
  static constexpr int TRIP = KM1 == 8 ? 64 : 224;  // whole phase periods
  static constexpr int NR = KM1 == 8 ? 4 : 7;       // divides the trip's half blocks
  float pm[R];
  uint32_t acc[R];
  float q[P][R];            // branch metrics of the stages ahead
  const float* tp[KM1][R];  // table entry of row 0
  float* bmt;               // 32 rows: stage t in row t mod 32
  float lr[NR][BETA];       // soft values of stage (lane & 15) of the half blocks ahead
  const In* llr;
  uint8_t* sv;              // survivor bytes of the frame, plus this lane's first position
  int S, lane;
  uint64_t bad;             // a soft value for wf_slow was seen
  float* xch;               // WPF > 1: two exchange buffers of the frame
  int fw, xb;
  __device__ __forceinline__ void load(float (&dst)[BETA], int tb) {
    const int64_t t = min(tb + (lane & 15), S - 1);  // past the end: not used
#pragma unroll
    for (int b = 0; b < BETA; ++b) dst[b] = (float)llr[t * BETA + b];
  }
};

// Table rows of a half block (half: 0 or 1): stage (lane & 15), four patterns
// per lane, bits 2 and 3 of the pattern being bits 4 and 5 of the lane (rates 1/2
// and 1/3: some lanes write alike).  With whole rows per lane, each written by
// four lanes, rate 1/4 frames over four wavefronts took 1.6 times as long (K =
// 9, 4096 of 4096 bits, forward: 1584 us, 977 now).
template <int KM1, int DT, int BETA, int WPF>
__device__ __forceinline__ void wf_table(Wf<KM1, DT, BETA, WPF>& F, const float (&lr)[BETA],
                                         int half) {
  constexpr int NP = 1 << BETA;
  float mag = 0.0f;
  float* row = F.bmt + (16 * half + (F.lane & 15)) * NP;
  float4 w;
#pragma unroll
  for (int p = 0; p < 2; ++p) {
    float v = 0.0f;
#pragma unroll
    for (int b = 0; b < 2; ++b) v += ((p >> b) & 1) ? -lr[b] : lr[b];
    if constexpr (BETA == 2) {
      row[p] = v;
      row[NP - 1 - p] = -v;
    } else {
      (p ? w.y : w.x) = v;
      (p ? w.z : w.w) = -v;
    }
  }
  if constexpr (BETA > 2) {
#pragma unroll
    for (int b = 2; b < BETA; ++b) {
      const uint32_t sign = (uint32_t)F.lane << (29 - b) & 0x80000000u;
      const float x = __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, lr[b]) ^ sign);
      w.x += x;
      w.y += x;
      w.z += x;
      w.w += x;
    }
    *(float4*)(row + ((F.lane >> 2) & (NP - 4))) = w;
  }
#pragma unroll
  for (int b = 0; b < BETA; ++b) mag += __builtin_fabsf(lr[b]);
  F.bad |= __builtin_amdgcn_ballot_w64(!(mag < 0x1p90f));
}

// Whether register r's metric is read at phase q: between registers only
// that of the even one (the odd new state has the opposite).
template <int R, int Q>
constexpr bool wf_reads(int r) {
  return !(Q >= 6 && (1 << (Q - 6)) < R) || !(r & (1 << (Q - 6)));
}

template <int KM1, int DT, int BETA, int WPF, int K>
__device__ __forceinline__ void wf_fetch(Wf<KM1, DT, BETA, WPF>& F) {
  using W = Wf<KM1, DT, BETA, WPF>;
#pragma unroll
  for (int r = 0; r < W::R; ++r)
    if (wf_reads<W::R, K % KM1>(r)) F.q[K % W::P][r] = F.tp[K % KM1][r][(K % 32) * W::NP];
}

// One stage at phase Q with branch metrics m.
template <int KM1, int DT, int BETA, int WPF, int Q>
__device__ __forceinline__ void wf_stage(Wf<KM1, DT, BETA, WPF>& F,
                                         const float (&m)[Wf<KM1, DT, BETA, WPF>::R]) {
  constexpr int R = Wf<KM1, DT, BETA, WPF>::R;
  float nv[R];
  uint32_t t[R];
  if constexpr (Q >= 6 && (1 << (Q - 6)) >= R) {
    // a wavefront bit: as in stage()
    constexpr int wb = (1 << (Q - 6)) / R;
    float* mine = F.xch + (WPF * F.xb + F.fw) * (64 * R) + F.lane;
    const float* theirs = F.xch + (WPF * F.xb + (F.fw ^ wb)) * (64 * R) + F.lane;
#pragma unroll
    for (int r = 0; r < R; ++r) mine[64 * r] = F.pm[r];
    frame_sync<true>();
    const bool odd = (F.fw & wb) != 0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const float other = theirs[64 * r];
      const float ce = (odd ? other : F.pm[r]) + m[r], co = (odd ? F.pm[r] : other) - m[r];
      nv[r] = rot::vmax(ce, co);
      t[r] = rot::diff_bits(ce, co);
    }
    F.xb ^= 1;
  } else if constexpr (Q >= 6) {
    constexpr int rb = 1 << (Q - 6);
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int re = r & ~rb, ro = r | rb;
      const float ce = (r & rb) ? F.pm[re] - m[re] : F.pm[re] + m[re];
      const float co = (r & rb) ? F.pm[ro] + m[re] : F.pm[ro] - m[re];
      nv[r] = rot::vmax(ce, co);
      t[r] = rot::diff_bits(ce, co);
    }
  } else if constexpr (rot::own_partner<Q>) {
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const float cp = rot::partner_fetch_valu<Q, 0>(F.pm[r]) - m[r];
      const float co = F.pm[r] + m[r];
      nv[r] = rot::max_and_diff<Q>(co, cp, t[r]);
    }
  } else {
#pragma unroll
    for (int r = 0; r < R; ++r) {
      float ce, co;
      if constexpr (Q < 2) {
        float e, o;
        rot::pair_fetch_valu<Q, 0>(F.pm[r], e, o);
        ce = e + m[r];
        co = o - m[r];
      } else {
        const int c0 = Ty<DT>::bits(F.pm[r] + m[r]), c1 = Ty<DT>::bits(F.pm[r] - m[r]);
        if constexpr (Q == 4) {
          const auto s = __builtin_amdgcn_permlane16_swap(c0, c1, false, false);
          ce = Ty<DT>::from(s[0]);
          co = Ty<DT>::from(s[1]);
        } else {
          const auto s = __builtin_amdgcn_permlane32_swap(c0, c1, false, false);
          ce = Ty<DT>::from(s[0]);
          co = Ty<DT>::from(s[1]);
        }
      }
      nv[r] = rot::vmax(ce, co);
      t[r] = rot::diff_bits(ce, co);
    }
  }
#pragma unroll
  for (int r = 0; r < R; ++r) {
    F.pm[r] = nv[r];
    F.acc[r] = rot::push_sign(F.acc[r], t[r]);
  }
}

// Stage K of a trip from t0.
template <int KM1, int DT, int BETA, int WPF, int K>
__device__ __forceinline__ void wf_step(Wf<KM1, DT, BETA, WPF>& F, int t0) {
  using W = Wf<KM1, DT, BETA, WPF>;
  if constexpr (K % 16 == 0) {
    constexpr int h = K / 16 + 1;  // the next half block
    auto& lr = F.lr[h % W::NR];
    wf_table(F, lr, h & 1);
    F.load(lr, t0 + 16 * (h + W::NR));
    frame_sync<false>();
  }
  float m[W::R];
#pragma unroll
  for (int r = 0; r < W::R; ++r) m[r] = F.q[K % W::P][r];
  wf_fetch<KM1, DT, BETA, WPF, K + W::P>(F);
  wf_stage<KM1, DT, BETA, WPF, K % KM1>(F, m);
  if constexpr (K % 32 == 31)
    store_block<KM1, W::R>(F.sv + (int64_t)((t0 + K) >> 5) * (4 * W::NS), F.acc);
}

template <int KM1, int DT, int BETA, int WPF, int K>
__device__ __forceinline__ void wf_trip(Wf<KM1, DT, BETA, WPF>& F, int t0) {
  if constexpr (K < Wf<KM1, DT, BETA, WPF>::TRIP) {
    wf_step<KM1, DT, BETA, WPF, K>(F, t0);
    wf_trip<KM1, DT, BETA, WPF, K + 1>(F, t0);
  }
}

// The last, partial trip: n stages from t0 (the decisions since the last
// whole block stay in acc).
template <int KM1, int DT, int BETA, int WPF, int K>
__device__ __forceinline__ void wf_tail(Wf<KM1, DT, BETA, WPF>& F, int t0, int n) {
  if constexpr (K < Wf<KM1, DT, BETA, WPF>::TRIP - 1) {
    if (K < n) {
      wf_step<KM1, DT, BETA, WPF, K>(F, t0);
      wf_tail<KM1, DT, BETA, WPF, K + 1>(F, t0, n);
    }
  }
}

// The frame's stages from t0 (a multiple of 32) on with compare and select,
// for soft values that bring NaNs or infinities.
template <int KM1, int DT, int BETA, int WPF>
__device__ __forceinline__ void wf_slow(Wf<KM1, DT, BETA, WPF>& F, const DevCode& c, int t0) {
  using W = Wf<KM1, DT, BETA, WPF>;
  Wave<DT, W::R> S;
#pragma unroll
  for (int r = 0; r < W::R; ++r) S.pm[r] = F.pm[r];
  S.xch = F.xch;
  S.nw = WPF;
  S.fw = F.fw;
  S.xb = F.xb;
  int pat[KM1][W::R];
  patterns<KM1, DT, W::R>(pat, c, F.lane, F.fw);
#pragma unroll 1
  for (int tb = t0; tb < F.S; tb += 32) {
    for (int half = 0; half < 2; ++half) {
      F.load(F.lr[0], tb + 16 * half);
      frame_sync<false>();
      wf_table(F, F.lr[0], half);
    }
    frame_sync<false>();
    const int n = min(32, F.S - tb);
#pragma unroll
    for (int r = 0; r < W::R; ++r) S.acc[r] = 0;
#pragma unroll 1
    for (int k = 0; k < n; ++k)
      stage_dyn<KM1, DT, W::R, W::NP, 0>(S, F.bmt + k * W::NP, pat, (tb + k) % KM1);
#pragma unroll
    for (int r = 0; r < W::R; ++r) S.acc[r] <<= 32 - n;
    store_block<KM1, W::R>(F.sv + (int64_t)(tb >> 5) * (4 * W::NS), S.acc);
  }
#pragma unroll
  for (int r = 0; r < W::R; ++r) F.pm[r] = S.pm[r];
}

}  // namespace wide

// One unit (whole item) per wavefront, or per workgroup of WPF wavefronts.
template <int KM1, int DT, int BETA, int WPF>
__global__ __launch_bounds__(64 * (WPF == 1 ? wide::kWideWaves : WPF), (1 << (KM1 - 6)) / WPF >= 4 ? 3 : 4) void k_fwd_wf(
    const DevCode* __restrict__ codes, const Item* __restrict__ items,
    const SplitUnit* __restrict__ units, int n_units, const void* __restrict__ llr_v,
    uint64_t* __restrict__ surv, float* metric, int32_t* end_out, int32_t* item_end) {
  using namespace wide;
  using W = Wf<KM1, DT, BETA, WPF>;
  constexpr int R = W::R, NS = W::NS;
  constexpr int kWaves = WPF == 1 ? kWideWaves : WPF;
  constexpr int FPB = WPF == 1 ? kWideWaves : 1;  // frames per workgroup
  __shared__ WfTable<BETA> bmt_all[kWaves];
  __shared__ float xpm_all[FPB][NS];
  __shared__ float xch_all[WPF > 1 ? 2 * WPF * 64 * R : 1];
  __shared__ float red_v[WPF];
  __shared__ int red_s[WPF];
  const int wid = threadIdx.x >> 6;
  const int lane = threadIdx.x & 63;
  const int fw = WPF == 1 ? 0 : wid;  // wavefront within the frame
  const int u = WPF == 1 ? blockIdx.x * kWideWaves + wid : blockIdx.x;
  // every wavefront of a frame leaves together: the barriers are per frame
  if (u >= n_units) return;
  const Item it = items[units[u].first];
  const DevCode c = codes[it.code];
  W F;
  F.S = __builtin_amdgcn_readfirstlane(it.n_stages);
  F.lane = lane;
  F.fw = fw;
  F.llr = (const typename Ty<DT>::In*)llr_v + it.llr_off;
  F.sv = (uint8_t*)(surv + it.surv_off) + 64 * R * fw + lane;
  F.bmt = bmt_all[wid].w;
  F.xch = xch_all;
  F.xb = 0;
  F.bad = 0;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    F.pm[r] = (it.start_known && (R * fw + r != 0 || lane != 0)) ? Ty<DT>::unreachable() : 0.0f;
    F.acc[r] = 0;
  }
#pragma unroll
  for (int q = 0; q < KM1; ++q) {
#pragma unroll
    for (int r = 0; r < R; ++r) {
      // as in the K <= 7 kernel; between registers or wavefronts: the even
      // previous state's branch into the new state
      const int p = 64 * (R * fw + r) + lane;
      const int j = rotr(p, (q + 1) % KM1, KM1);
      const int ie = (j << 1) & (NS - 1);
      const int own = rotr(p, q, KM1);
      F.tp[q][r] = F.bmt + (q == 2 || q == 3   ? branch_out(c, ie, 0)
                            : q == 4 || q == 5 ? branch_out(c, own, 0)
                                               : branch_out(c, ie, j >> (KM1 - 1)));
    }
  }
  if (F.S > 0) {
#pragma unroll
    for (int k = 0; k < W::NR; ++k) F.load(F.lr[k], 16 * k);
    wf_table(F, F.lr[0], 0);
    F.load(F.lr[0], 16 * W::NR);
    frame_sync<false>();
    [&]<int... K>(std::integer_sequence<int, K...>) {
      (wf_fetch<KM1, DT, BETA, WPF, K>(F), ...);
    }(std::make_integer_sequence<int, W::P>());
    int t0 = 0;
    float pm0[R];  // metrics entering the trip from t0
#pragma unroll
    for (int r = 0; r < R; ++r) pm0[r] = F.pm[r];
    // (only where wavefronts share SIMDs: K = 9, 1500 frames of 3000 bits 268
    // -> 250 us, K = 8, 4096 of 2000 180 -> 175)
    const int slot = WPF == 1 && gridDim.x > kComputeUnits ? wave_slot() : -1;
    for (; t0 + W::TRIP <= F.S && F.bad == 0; t0 += W::TRIP) {
      if (slot >= 0) fair_share(slot, t0 / W::TRIP);
#pragma unroll
      for (int r = 0; r < R; ++r) pm0[r] = F.pm[r];
      wf_trip<KM1, DT, BETA, WPF, 0>(F, t0);
    }
    if (F.bad != 0) {
      t0 = max(t0 - W::TRIP, 0);
    } else {
#pragma unroll
      for (int r = 0; r < R; ++r) pm0[r] = F.pm[r];
      wf_tail<KM1, DT, BETA, WPF, 0>(F, t0, F.S - t0);
      const int rem = F.S & 31;
      if (rem) {
        uint32_t a[R];
#pragma unroll
        for (int r = 0; r < R; ++r) a[r] = F.acc[r] << (32 - rem);
        store_block<KM1, R>(F.sv + (int64_t)(F.S >> 5) * (4 * NS), a);
      }
    }
    if (F.bad != 0) {
      // the trip in which they were seen, again
#pragma unroll
      for (int r = 0; r < R; ++r) F.pm[r] = pm0[r];
      if constexpr (WPF > 1) frame_sync<true>();
      wf_slow(F, c, t0);
    }
  }
  int js;
  const float vj = end_state<KM1, DT, R, WPF>(F.pm, F.S, lane, fw, it.end_state,
                                              xpm_all[WPF == 1 ? wid : 0], red_v, red_s, js);
  if (lane == 0 && fw == 0) {
    item_end[it.slot] = js;
    if (it.frame >= 0 && end_out) end_out[it.frame] = js;
    if (it.frame >= 0 && metric) metric[it.frame] = vj;
  }
}

template <int DT>
hipError_t wf_launch(int K, int beta, int wpf, const DevCode* codes, const Item* items,
                     const SplitUnit* units, int n_units, const void* llr, uint64_t* surv,
                     void* metric, int32_t* end_out, int32_t* item_end, hipStream_t st) {
  const int fpb = wpf == 1 ? wide::kWideWaves : 1;
  const dim3 grid((n_units + fpb - 1) / fpb), block(64 * (wpf == 1 ? wide::kWideWaves : wpf));
#define MV_WF(K, B, W)                                                                        \
  case K * 64 + B * 8 + W:                                                                    \
    hipLaunchKernelGGL((k_fwd_wf<K - 1, DT, B, W>), grid, block, 0, st, codes, items, units,  \
                       n_units, llr, surv, (float*)metric, end_out, item_end);                \
    break
  switch (K * 64 + beta * 8 + wpf) {
    MV_WF(8, 2, 1); MV_WF(8, 3, 1); MV_WF(8, 4, 1);
    MV_WF(9, 2, 1); MV_WF(9, 3, 1); MV_WF(9, 4, 1);
    MV_WF(8, 2, 2); MV_WF(8, 3, 2); MV_WF(8, 4, 2);
    MV_WF(9, 2, 2); MV_WF(9, 3, 2); MV_WF(9, 4, 2);
    MV_WF(9, 2, 4); MV_WF(9, 3, 4); MV_WF(9, 4, 4);
    default: return hipErrorInvalidValue;
  }
#undef MV_WF
  return hipGetLastError();
}

}  // namespace mivit

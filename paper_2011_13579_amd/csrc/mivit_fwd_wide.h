// Radix-2 forward procedure for K = 8 and 9 (128 and 256 states): one
// wavefront per frame (float frames: one, two or four), R = 2^(K-1)/64 states
// per lane held in registers.  Shared parts of the int8 kernels
// (mivit_fwd_wide.hip) and the float kernel (mivit_fwd_wide_float.h).
//
// The state-to-position map rotates as in the K <= 7 kernel: at time t the
// state s sits at position rotl_n(s, t mod n), n = K-1, and position p is
// register p >> 6 of lane p & 63.  At stage t (phase q = t mod n) both
// previous states (Eq. (radix2:S): 2f and 2f+1) of the state at position p
// sit at the positions p with bit q cleared and set, and the new state stays
// at p.  For q < 6 that is an exchange between lanes, done for each of the R
// registers: DPP quad permutations fetch both previous metrics for bits 0
// and 1, v_permlane16/32_swap for bits 4 and 5.  For bits 2 and 3, float
// metrics stay in the VALU: a lane keeps its own previous state's metric and
// fetches its partner's (lane ^ 4: row half-mirror then quad reverse; lane ^
// 8: row rotate by 8); integer metrics fetch both through ds_swizzle, which
// measured faster for them.  For q >= 6 the two previous states are two
// registers of the same lane and nothing moves.  The R registers are independent dependency
// chains, which keeps a lone wavefront busy.
//
// Branch metrics: Eq. (BM) for the even previous state on the new state's
// input; by the corollary of §IV the odd previous state's branch has the
// opposite value.  A per-wavefront LDS table holds the 2^beta pattern values
// of each stage of a 32-stage block.
//
// Decisions: d = 1 when the odd previous state wins (strict, so a tie keeps
// the even, lower-index one).  Every position shifts its decision into a
// 32-bit word; every 32 stages its four bytes go out: per group of 8 stages, 2^(K-1) bytes, byte p
// holding position p's decisions with stage 8g + i at bit 7 - i.  A group of
// 8 stages is then 64 (K = 9) or 32 (K = 8) words, the unit the traceback
// stages through LDS.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "mivit_device.h"

namespace mivit {

namespace wide {

template <int DT>
struct Ty;
template <>
struct Ty<0> {
  static constexpr bool kInt = false;
  using T = float;
  using In = float;
  __device__ static float unreachable() { return -__builtin_inff(); }
  __device__ static int bits(float x) { return __builtin_bit_cast(int, x); }
  __device__ static float from(int x) { return __builtin_bit_cast(float, x); }
};
template <>
struct Ty<1> {
  static constexpr bool kInt = true;
  using T = int;
  using In = int8_t;
  __device__ static int unreachable() { return -(1 << 29); }
  __device__ static int bits(int x) { return x; }
  __device__ static int from(int x) { return x; }
};
template <>
struct Ty<2> : Ty<0> {
  using In = _Float16;
};

__device__ __forceinline__ int parity(uint32_t x) { return __popc(x) & 1; }

__device__ __forceinline__ int branch_out(const DevCode& c, int i, int u) {
  const uint32_t reg = ((uint32_t)u << (c.K - 1)) | (uint32_t)i;
  int w = 0;
#pragma unroll
  for (int b = 0; b < 4; ++b)
    if (b < c.beta) w |= parity(c.gen[b] & reg) << b;
  return w;
}

__device__ __forceinline__ int rotl(int x, int r, int n) {
  return r == 0 ? x : (((x << r) | (x >> (n - r))) & ((1 << n) - 1));
}
__device__ __forceinline__ int rotr(int x, int r, int n) { return rotl(x, (n - r) % n, n); }

// Metrics of the even and odd previous states across lane bit Q (Q < 6).
template <int Q, int DT>
__device__ __forceinline__ void pair_fetch(typename Ty<DT>::T x, typename Ty<DT>::T& e,
                                           typename Ty<DT>::T& o) {
  const int xi = Ty<DT>::bits(x);
  int ei, oi;
  if constexpr (Q == 0) {
    ei = __builtin_amdgcn_mov_dpp(xi, 0xA0, 0xF, 0xF, true);  // quad_perm [0,0,2,2]
    oi = __builtin_amdgcn_mov_dpp(xi, 0xF5, 0xF, 0xF, true);  // quad_perm [1,1,3,3]
  } else if constexpr (Q == 1) {
    ei = __builtin_amdgcn_mov_dpp(xi, 0x44, 0xF, 0xF, true);  // quad_perm [0,1,0,1]
    oi = __builtin_amdgcn_mov_dpp(xi, 0xEE, 0xF, 0xF, true);  // quad_perm [2,3,2,3]
  } else if constexpr (Q <= 3) {
    // bit-mask mode within 32 lanes: lane' = (lane & and_mask) | or_mask
    ei = __builtin_amdgcn_ds_swizzle(xi, 0x1F & ~(1 << Q));
    oi = __builtin_amdgcn_ds_swizzle(xi, 0x1F | ((1 << Q) << 5));
  } else if constexpr (Q == 4) {
    // even rows of 16 to every row, odd rows to every row
    const auto r = __builtin_amdgcn_permlane16_swap(xi, xi, false, false);
    ei = r[0];
    oi = r[1];
  } else {
    const auto r = __builtin_amdgcn_permlane32_swap(xi, xi, false, false);
    ei = r[0];
    oi = r[1];
  }
  e = Ty<DT>::from(ei);
  o = Ty<DT>::from(oi);
}

// Stages at lane bits 2 and 3 in own/partner form (float metrics).
template <int DT, int Q>
constexpr bool own_partner() {
  return (Q == 2 || Q == 3) && !Ty<DT>::kInt;
}

// Metric of the partner lane (lane ^ 2^Q) for Q = 2, 3.
template <int Q, int DT>
__device__ __forceinline__ typename Ty<DT>::T partner_fetch(typename Ty<DT>::T x) {
  const int xi = Ty<DT>::bits(x);
  int pi;
  if constexpr (Q == 2) {
    const int hm = __builtin_amdgcn_mov_dpp(xi, 0x141, 0xF, 0xF, true);  // row_half_mirror: ^7
    pi = __builtin_amdgcn_mov_dpp(hm, 0x1B, 0xF, 0xF, true);            // quad_perm [3,2,1,0]: ^3
  } else {
    pi = __builtin_amdgcn_mov_dpp(xi, 0x128, 0xF, 0xF, true);  // row_ror:8
  }
  return Ty<DT>::from(pi);
}

template <int DT, int R>
struct Wave {
  using T = typename Ty<DT>::T;
  T pm[R];           // metric of the state at position 64 (R w + r) + lane
  uint32_t acc[R];   // decisions of that position in the current block
  uint32_t pend[R];  // the previous block's decision words, not yet stored
  // several wavefronts per frame: LDS exchange area of the frame, the
  // number of wavefronts, this one's index w in the frame, and the exchange
  // buffer in use
  T* xch;
  int nw, fw, xb;
};

// All wavefronts of a frame at one point, LDS writes before it visible to
// LDS reads after it.  One wavefront per frame: program order suffices;
// several (kWorkgroup): the frame is the workgroup, a barrier.
template <bool kWorkgroup>
__device__ __forceinline__ void frame_sync() {
  if constexpr (!kWorkgroup) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  } else {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
  }
}


// The larger of two metrics; of a number and a NaN, the number.  (Floats come
// here only from the loop for soft values that bring NaNs or infinities, and
// the decision beside it compares, so a NaN candidate never wins.)
__device__ __forceinline__ float tmax(float a, float b) { return __builtin_fmaxf(a, b); }
__device__ __forceinline__ int tmax(int a, int b) { return a > b ? a : b; }

// push_decision for every register of a stage: one wait state pair for all
// of them (a VALU-written SGPR read as carry needs two).
template <int R>
__device__ __forceinline__ void push_decisions(uint32_t (&acc)[R], const uint64_t (&d)[R]) {
  if constexpr (R == 4) {
    uint64_t c0, c1, c2, c3;
    asm("s_nop 1\n\t"
        "v_addc_co_u32_e64 %0, %4, %0, %0, %8\n\t"
        "v_addc_co_u32_e64 %1, %5, %1, %1, %9\n\t"
        "v_addc_co_u32_e64 %2, %6, %2, %2, %10\n\t"
        "v_addc_co_u32_e64 %3, %7, %3, %3, %11"
        : "+v"(acc[0]), "+v"(acc[1]), "+v"(acc[2]), "+v"(acc[3]), "=s"(c0), "=s"(c1), "=s"(c2),
          "=s"(c3)
        : "s"(d[0]), "s"(d[1]), "s"(d[2]), "s"(d[3]));
  } else {
#pragma unroll
    for (int r = 0; r < R; ++r) acc[r] = push_decision(acc[r], d[r]);
  }
}

// One stage at phase Q; bm[r] the branch metric of position 64r + lane: of
// its even previous state, or in own/partner form of its own previous state
// (the state at position 64r + lane before the stage).  Own/partner form: the
// candidates are own + bm and partner - bm in every lane (by the corollary
// the other previous state's branch has the opposite value); the odd
// previous state won when partner > own where the lane's bit Q is 0 and
// own > partner where it is 1, strictly, so a tie keeps the even state.
template <int KM1, int DT, int R, int Q>
__device__ __forceinline__ void stage(Wave<DT, R>& W, const typename Ty<DT>::T (&bm)[R]) {
  using T = typename Ty<DT>::T;
  T nv[R];
  uint64_t d[R];  // lanes whose odd previous state won
  if constexpr (Q >= 6 && (1 << (Q - 6)) >= R) {
    // bit Q is bit wb of the wavefront index (several per frame): the
    // wavefronts with that bit clear hold the even previous states, their
    // partners (index ^ wb) the odd ones, at the same register and lane;
    // each writes its metrics to the exchange buffer and reads its partner's
    constexpr int wb = (1 << (Q - 6)) / R;
    const int lane = threadIdx.x & 63;
    const int nw = W.nw;
    T* mine = W.xch + (nw * W.xb + W.fw) * (64 * R);
    const T* theirs = W.xch + (nw * W.xb + (W.fw ^ wb)) * (64 * R);
#pragma unroll
    for (int r = 0; r < R; ++r) mine[64 * r + lane] = W.pm[r];
    frame_sync<true>();
    const bool odd = (W.fw & wb) != 0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const T other = theirs[64 * r + lane];
      const T e = odd ? other : W.pm[r], o = odd ? W.pm[r] : other;
      const T ce = e + bm[r], co = o - bm[r];
      nv[r] = tmax(ce, co);
      d[r] = __builtin_amdgcn_ballot_w64(co > ce);
    }
    // double buffered: the next exchange writes the other buffer, and the
    // one after it comes after a barrier that follows these reads
    W.xb ^= 1;
  } else if constexpr (own_partner<DT, Q>()) {
    // lanes with bit Q set hold the odd previous state
    constexpr uint64_t odd = Q == 2 ? 0xF0F0F0F0F0F0F0F0ull : 0xFF00FF00FF00FF00ull;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const T cp = partner_fetch<Q, DT>(W.pm[r]) - bm[r];
      const T co = W.pm[r] + bm[r];
      nv[r] = tmax(cp, co);
      d[r] = (__builtin_amdgcn_ballot_w64(cp > co) & ~odd) |
             (__builtin_amdgcn_ballot_w64(co > cp) & odd);
    }
  } else if constexpr (Q < 6) {
#pragma unroll
    for (int r = 0; r < R; ++r) {
      T e, o;
      pair_fetch<Q, DT>(W.pm[r], e, o);
      const T ce = e + bm[r], co = o - bm[r];
      nv[r] = tmax(ce, co);
      d[r] = __builtin_amdgcn_ballot_w64(co > ce);
    }
  } else {
    constexpr int rb = 1 << (Q - 6);
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int re = r & ~rb, ro = r | rb;
      const T ce = W.pm[re] + bm[r], co = W.pm[ro] - bm[r];
      nv[r] = tmax(ce, co);
      d[r] = __builtin_amdgcn_ballot_w64(co > ce);
    }
  }
#pragma unroll
  for (int r = 0; r < R; ++r) W.pm[r] = nv[r];
  push_decisions<R>(W.acc, d);
}

// A stage whose phase is only known at run time (the last, partial block).
template <int KM1, int DT, int R, int NP, int Q>
__device__ __forceinline__ void stage_dyn(Wave<DT, R>& W, const typename Ty<DT>::T* bmrow,
                                          const int (&pat)[KM1][R], int q) {
  if constexpr (Q < KM1) {
    if (q == Q) {
      typename Ty<DT>::T bm[R];
#pragma unroll
      for (int r = 0; r < R; ++r) bm[r] = bmrow[pat[Q][r]];
      stage<KM1, DT, R, Q>(W, bm);
    } else {
      stage_dyn<KM1, DT, R, NP, Q + 1>(W, bmrow, pat, q);
    }
  }
}

__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Store one block's decision words: four groups of 8 stages, group g of the
// block being byte 3 - g of the word.
template <int KM1, int R>
__device__ __forceinline__ void store_block(uint8_t* dst, const uint32_t (&a)[R]) {
  constexpr int NS = 1 << KM1;
#pragma unroll
  for (int r = 0; r < R; ++r) {
#pragma unroll
    for (int g = 0; g < 4; ++g) dst[g * NS + 64 * r] = (uint8_t)(a[r] >> (24 - 8 * g));
  }
}

constexpr int gcd_c(int a, int b) { return b == 0 ? a : gcd_c(b, a % b); }

// Table offset (pattern) of position 64 (R w + r) + lane at each phase, for
// stage(): the even previous state's branch into the state held there after
// the stage, or in own/partner form the branch of the previous state at p
// (odd when bit q of p is set).
template <int KM1, int DT, int R>
__device__ __forceinline__ void patterns(int (&pat)[KM1][R], const DevCode& c, int lane, int fw) {
#pragma unroll
  for (int q = 0; q < KM1; ++q) {
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int j = rotr(64 * (R * fw + r) + lane, (q + 1) % KM1, KM1);
      const bool op = (q == 2 || q == 3) && !Ty<DT>::kInt;
      const int own = op ? ((lane >> q) & 1) : 0;
      pat[q][r] = branch_out(c, ((j << 1) | own) & ((1 << KM1) - 1), j >> (KM1 - 1));
    }
  }
}

// The final state js (end, or the best state for end < 0, ties to the lowest
// index; state 0 when no metric compares, all being NaN) and its metric.
// Position p holds state rotr(p, S mod (K-1)); xpm: 2^(K-1) words of LDS,
// red_v, red_s: WPF words each.
template <int KM1, int DT, int R, int WPF>
__device__ __forceinline__ typename Ty<DT>::T end_state(const typename Ty<DT>::T (&pm)[R], int S,
                                                        int lane, int fw, int end,
                                                        typename Ty<DT>::T* xpm,
                                                        typename Ty<DT>::T* red_v, int* red_s,
                                                        int& js) {
  using T = typename Ty<DT>::T;
  constexpr int NS = 1 << KM1;
  T bv = Ty<DT>::unreachable();
  int bs = NS;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int s = rotr(64 * (R * fw + r) + lane, S % KM1, KM1);
    xpm[s] = pm[r];
    if (pm[r] > bv || (pm[r] == bv && s < bs)) {
      bv = pm[r];
      bs = s;
    }
  }
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const T ov = Ty<DT>::from(__shfl_xor(Ty<DT>::bits(bv), o));
    const int os = __shfl_xor(bs, o);
    if (ov > bv || (ov == bv && os < bs)) {
      bv = ov;
      bs = os;
    }
  }
  if constexpr (WPF > 1) {
    // the best of the wavefronts' best states, ties to the lower index
    if (lane == 0) {
      red_v[fw] = bv;
      red_s[fw] = bs;
    }
    frame_sync<true>();
#pragma unroll
    for (int k = 0; k < WPF; ++k) {
      const T ov = red_v[k];
      const int os = red_s[k];
      if (ov > bv || (ov == bv && os < bs)) {
        bv = ov;
        bs = os;
      }
    }
  } else {
    frame_sync<false>();
  }
  js = end >= 0 ? end : bs < NS ? bs : 0;
  return xpm[js];
}

constexpr int kWideWaves = 4;  // independent wavefronts (frames) per workgroup

}  // namespace wide

}  // namespace mivit

// Radix-2 forward procedure for K <= 7 with a rotating state-to-lane map.
//
// Eq. (radix2:S) pairs the previous states 2f and 2f+1 (differing in their
// LSB) into the states f and f + 2^(K-2) (differing in their MSB).  With n =
// K-1 state bits, let the state s live in lane rotl_n(s, t mod n) at time t.
// Then at stage t both previous states of the state in lane l sit in lanes
// l with bit (t mod n) cleared and set, and the new state stays in lane l: a
// butterfly is an exchange between two lanes that differ in one lane bit, and
// no data moves otherwise.  The default form (MODE 2, fwd_rot_valu_wave)
// exchanges in the vector ALU; MODE 0 and 1 exchange through LDS swizzles.
//
// Branch metrics: by the corollary of §IV (MSB and LSB taps set) the two
// branches into a state carry opposite metrics, delta(2f+1 -> j) =
// -delta(2f -> j), so each lane reads one value per stage from a per-frame
// LDS table of Eq. (BM) over the 2^beta output patterns.
//
// Decisions: d = 1 when the odd previous state wins (strict comparison, so a
// tie keeps the even, lower-index one).  Each lane shifts its decision into a
// 32-bit word (bit 31 - (t mod 32) holds stage t); every 32 stages the words
// of a frame's lanes are stored together, word index = lane.
//
// One wavefront runs 64/2^(K-1) frames of equal length side by side.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "mivit_device.h"

namespace mivit {

namespace rot {

constexpr int gcd_c(int a, int b) { return b == 0 ? a : gcd_c(b, a % b); }

__device__ __forceinline__ int parity(uint32_t x) { return __popc(x) & 1; }

__device__ __forceinline__ int branch_out(const DevCode& c, int i, int u) {
  uint32_t reg = ((uint32_t)u << (c.K - 1)) | (uint32_t)i;
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

// Soft-value type DT (0: float32, 1: int8, 2: float16) and the metric
// arithmetic it runs in: float32 for both float types (a float16 value
// converts to float32 exactly), exact int32 with renormalisation for int8.
template <int DT>
struct Ty;
template <>
struct Ty<0> {
  static constexpr bool kInt = false;
  using T = float;
  using In = float;
  __device__ static float neg_unreachable() { return -__builtin_inff(); }
  __device__ static int bits(float x) { return __builtin_bit_cast(int, x); }
  __device__ static float from(int x) { return __builtin_bit_cast(float, x); }
};
template <>
struct Ty<1> {
  static constexpr bool kInt = true;
  using T = int;
  using In = int8_t;
  __device__ static int neg_unreachable() { return -(1 << 29); }
  __device__ static int bits(int x) { return x; }
  __device__ static int from(int x) { return x; }
};
template <>
struct Ty<2> : Ty<0> {
  using In = _Float16;
};

// Fetch the metrics of the even and odd previous states for lane bit Q.
template <int Q, int DT>
__device__ __forceinline__ void pair_fetch(typename Ty<DT>::T x, int addr_e, int addr_o,
                                           typename Ty<DT>::T& e, typename Ty<DT>::T& o) {
  const int xi = Ty<DT>::bits(x);
  int ei, oi;
  if constexpr (Q == 0) {
    ei = __builtin_amdgcn_mov_dpp(xi, 0xA0, 0xF, 0xF, true);  // quad_perm [0,0,2,2]
    oi = __builtin_amdgcn_mov_dpp(xi, 0xF5, 0xF, 0xF, true);  // quad_perm [1,1,3,3]
  } else if constexpr (Q == 1) {
    ei = __builtin_amdgcn_mov_dpp(xi, 0x44, 0xF, 0xF, true);  // quad_perm [0,1,0,1]
    oi = __builtin_amdgcn_mov_dpp(xi, 0xEE, 0xF, 0xF, true);  // quad_perm [2,3,2,3]
  } else if constexpr (Q <= 4) {
    // ds_swizzle bit-mask mode within 32 lanes: lane' = (lane & and) | or
    ei = __builtin_amdgcn_ds_swizzle(xi, 0x1F & ~(1 << Q));
    oi = __builtin_amdgcn_ds_swizzle(xi, 0x1F | ((1 << Q) << 5));
  } else {
    ei = __builtin_amdgcn_ds_bpermute(addr_e, xi);
    oi = __builtin_amdgcn_ds_bpermute(addr_o, xi);
  }
  e = Ty<DT>::from(ei);
  o = Ty<DT>::from(oi);
}

// Fetch the metric of the partner lane (lane XOR 2^Q).  XOR 1, 2 and 8 are
// single DPP patterns (fused by the compiler into the consuming subtract).
template <int Q, int DT>
__device__ __forceinline__ typename Ty<DT>::T partner_fetch(typename Ty<DT>::T x, int addr_p) {
  const int xi = Ty<DT>::bits(x);
  int pi;
  if constexpr (Q == 0) {
    pi = __builtin_amdgcn_mov_dpp(xi, 0xB1, 0xF, 0xF, true);  // quad_perm [1,0,3,2]
  } else if constexpr (Q == 1) {
    pi = __builtin_amdgcn_mov_dpp(xi, 0x4E, 0xF, 0xF, true);  // quad_perm [2,3,0,1]
  } else if constexpr (Q == 3) {
    pi = __builtin_amdgcn_mov_dpp(xi, 0x128, 0xF, 0xF, true);  // row_ror:8
  } else if constexpr (Q == 2 || Q == 4) {
    pi = __builtin_amdgcn_ds_swizzle(xi, 0x1F | ((1 << Q) << 10));  // xor mode
  } else {
    pi = __builtin_amdgcn_ds_bpermute(addr_p, xi);
  }
  return Ty<DT>::from(pi);
}

template <int KM1, int DT, int NP, int MODE>
struct Frame {
  using T = typename Ty<DT>::T;
  T pm;
  uint32_t acc;
  int pat_off[KM1];  // LDS word offset of this lane's pattern, per phase
  int addr_e, addr_o, addr_p;
  uint64_t bmask[KM1];  // lanes whose bit q is set, per phase q
};

// MODE 2 exchanges, per lane bit:
//   bits 0, 1  both previous-state metrics by DPP quad permutations
//   bit 2      partner (lane ^ 4) = quad reverse of the row half-mirror (two DPPs)
//   bit 3      partner (lane ^ 8) = DPP row rotate by 8
//   bits 4, 5  v_permlane16_swap / v_permlane32_swap
template <int Q>
constexpr bool own_partner = Q == 2 || Q == 3;

template <int Q, int DT>
__device__ __forceinline__ void pair_fetch_valu(typename Ty<DT>::T x, typename Ty<DT>::T& e,
                                                typename Ty<DT>::T& o) {
  const int xi = Ty<DT>::bits(x);
  int ei, oi;
  if constexpr (Q == 0) {
    ei = __builtin_amdgcn_mov_dpp(xi, 0xA0, 0xF, 0xF, true);
    oi = __builtin_amdgcn_mov_dpp(xi, 0xF5, 0xF, 0xF, true);
  } else if constexpr (Q == 1) {
    ei = __builtin_amdgcn_mov_dpp(xi, 0x44, 0xF, 0xF, true);
    oi = __builtin_amdgcn_mov_dpp(xi, 0xEE, 0xF, 0xF, true);
  } else if constexpr (Q == 4) {
    auto r = __builtin_amdgcn_permlane16_swap(xi, xi, false, false);
    ei = r[0];
    oi = r[1];
  } else {
    auto r = __builtin_amdgcn_permlane32_swap(xi, xi, false, false);
    ei = r[0];
    oi = r[1];
  }
  e = Ty<DT>::from(ei);
  o = Ty<DT>::from(oi);
}

template <int Q, int DT>
__device__ __forceinline__ typename Ty<DT>::T partner_fetch_valu(typename Ty<DT>::T x) {
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

template <typename T>
__device__ __forceinline__ T tmax(T a, T b) {
  return a > b ? a : b;
}

// One stage at phase Q, own/partner form.  The lane keeps its own previous
// state's metric and fetches its partner's.  With m0 the Eq. (BM) value of
// the even previous state on input 0, the candidate through the lane's own
// previous state is own + m0 and through the partner's is partner - m0, in
// every lane (the corollary flips the sign once for the odd state and once
// for input 1).  The new metric is the larger one; the decision "the odd
// previous state won" is partner > own where the lane's bit Q is 0 (partner
// odd) and own > partner where it is 1 (own odd), strict either way, so a tie
// keeps the even state.
template <int KM1, int DT, int NP, int MODE, int Q>
__device__ __forceinline__ void stage_op(Frame<KM1, DT, NP, MODE>& F, typename Ty<DT>::T m0) {
  using T = typename Ty<DT>::T;
  const T cp = partner_fetch<Q, DT>(F.pm, F.addr_p) - m0;
  const T co = F.pm + m0;
  F.pm = tmax(co, cp);
  const uint64_t g1 = __builtin_amdgcn_ballot_w64(cp > co);
  const uint64_t g2 = __builtin_amdgcn_ballot_w64(co > cp);
  const uint64_t d = (g1 & ~F.bmask[Q]) | (g2 & F.bmask[Q]);
  F.acc = push_decision(F.acc, d);
}

// One stage at phase Q: add, compare, select, record.
template <int KM1, int DT, int NP, int MODE, int Q>
__device__ __forceinline__ void stage(Frame<KM1, DT, NP, MODE>& F, typename Ty<DT>::T bm) {
  using T = typename Ty<DT>::T;
  T e, o;
  pair_fetch<Q, DT>(F.pm, F.addr_e, F.addr_o, e, o);
  const T ce = e + bm;  // even previous state, Eq. (PM) candidate
  const T co = o - bm;  // odd previous state: opposite branch metric
  const bool d = co > ce;
  F.pm = d ? co : ce;
  F.acc = push_decision(F.acc, __builtin_amdgcn_ballot_w64(d));
}

template <int KM1, int DT, int NP, int MODE, int Q>
__device__ __forceinline__ void stage_any(Frame<KM1, DT, NP, MODE>& F, typename Ty<DT>::T bm) {
  if constexpr (MODE == 1)
    stage_op<KM1, DT, NP, MODE, Q>(F, bm);
  else
    stage<KM1, DT, NP, MODE, Q>(F, bm);
}

template <int KM1, int DT, int NP, int MODE, int P0, int K0>
__device__ __forceinline__ void stages_full(Frame<KM1, DT, NP, MODE>& F,
                                            const typename Ty<DT>::T* bmv) {
  if constexpr (K0 < 32) {
    stage_any<KM1, DT, NP, MODE, (P0 + K0) % KM1>(F, bmv[K0]);
    stages_full<KM1, DT, NP, MODE, P0, K0 + 1>(F, bmv);
  }
}

// A stage whose phase is only known at run time (the last, partial block).
template <int KM1, int DT, int NP, int MODE, int Q>
__device__ __forceinline__ void stage_dyn(Frame<KM1, DT, NP, MODE>& F, const typename Ty<DT>::T* bmrow,
                                          int q) {
  if constexpr (Q < KM1) {
    if (q == Q) {
      stage_any<KM1, DT, NP, MODE, Q>(F, bmrow[F.pat_off[Q]]);
    } else {
      stage_dyn<KM1, DT, NP, MODE, Q + 1>(F, bmrow, q);
    }
  }
}

template <int KM1, int DT, int NP, int MODE, int P0>
__device__ __forceinline__ void block(Frame<KM1, DT, NP, MODE>& F, const typename Ty<DT>::T* bmt,
                                      int n) {
  using T = typename Ty<DT>::T;
  if (n == 32) {
    // this lane's branch metric of every stage of the block, read up front
    T bmv[32];
#pragma unroll
    for (int k = 0; k < 32; ++k) bmv[k] = bmt[k * NP + F.pat_off[(P0 + k) % KM1]];
    stages_full<KM1, DT, NP, MODE, P0, 0>(F, bmv);
  } else {
#pragma unroll 1
    for (int k = 0; k < n; ++k) stage_dyn<KM1, DT, NP, MODE, 0>(F, bmt + k * NP, (P0 + k) % KM1);
  }
}

// Order LDS traffic between the lanes of one wavefront.  LDS instructions of
// a wavefront execute in order, so a compiler-level fence at wavefront scope
// is enough; unlike a workgroup barrier it does not wait for the outstanding
// global loads that prefetch the next block.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Soft values of the stages a lane tabulates in one block: stages
// sl + k*2^(K-1) for k < max(1, 32/2^(K-1)).
template <int KM1, int DT, int BETA>
struct LlrRegs {
  static constexpr int NS = 1 << KM1;
  static constexpr int NSTG = NS >= 32 ? 1 : 32 / NS;
  typename Ty<DT>::T v[NSTG][BETA];
  __device__ __forceinline__ void load(const typename Ty<DT>::In* llr, int tb, int S, int sl,
                                       bool valid) {
#pragma unroll
    for (int k = 0; k < NSTG; ++k) {
      const int t = tb + sl + k * NS;
      const bool ok = valid && sl + k * NS < 32 && t < S;
#pragma unroll
      for (int b = 0; b < BETA; ++b)
        v[k][b] = ok ? (typename Ty<DT>::T)llr[(int64_t)t * BETA + b] : (typename Ty<DT>::T)0;
    }
  }
};

// State shared by the blocks of one wavefront.
template <int KM1, int DT, int BETA, int MODE>
struct BlockCtx {
  Frame<KM1, DT, (1 << BETA), MODE>* F;
  typename Ty<DT>::T* bmt;
  const typename Ty<DT>::In* llr;
  uint32_t* sv;
  int64_t* offset;
  int* blk;
  int S, sl, lane;
  bool valid;
  LlrRegs<KM1, DT, BETA> lr;  // soft values of the current block, loaded a block ahead
};

// One block of up to 32 stages starting at tb, phase (32*BI) mod (K-1).
template <int KM1, int DT, int BETA, int MODE, int BI>
__device__ __forceinline__ void one_block(BlockCtx<KM1, DT, BETA, MODE>& bc, int tb) {
  using T = typename Ty<DT>::T;
  constexpr int NS = 1 << KM1, NP = 1 << BETA;
  constexpr int NSTG = LlrRegs<KM1, DT, BETA>::NSTG;
  const int n = min(32, bc.S - tb);
  // branch-metric table of this block: Eq. (BM) for every output pattern
#pragma unroll
  for (int k = 0; k < NSTG; ++k) {
    const int tt = bc.sl + k * NS;
    if (tt < 32) {
#pragma unroll
      for (int p = 0; p < NP / 2; ++p) {
        T v = (T)0;
#pragma unroll
        for (int b = 0; b < BETA; ++b) v += ((p >> b) & 1) ? -bc.lr.v[k][b] : bc.lr.v[k][b];
        bc.bmt[tt * NP + p] = v;
        bc.bmt[tt * NP + (NP - 1 - p)] = -v;
      }
    }
  }
  // the next block's soft values are read while this block runs
  bc.lr.load(bc.llr, tb + 32, bc.S, bc.sl, bc.valid);
  if constexpr (Ty<DT>::kInt) {
    if (tb > 0) {
      // renormalise by the metric of state 0 (always in the frame's lane 0)
      const T ref = __builtin_amdgcn_ds_bpermute((bc.lane & ~(NS - 1)) << 2, bc.F->pm);
      bc.F->pm -= ref;
      *bc.offset += ref;
    }
  }
  wave_sync();
  block<KM1, DT, NP, MODE, (32 * BI) % KM1>(*bc.F, bc.bmt, n);
  if (bc.valid) bc.sv[(int64_t)(*bc.blk) * NS + bc.sl] = bc.F->acc << (32 - n);
  bc.F->acc = 0;
  ++*bc.blk;
  wave_sync();
}

template <int KM1, int DT, int BETA, int MODE, int BI, int NB>
__device__ __forceinline__ void super_block(BlockCtx<KM1, DT, BETA, MODE>& bc, int t0) {
  if constexpr (BI < NB) {
    const int tb = t0 + 32 * BI;
    if (tb < bc.S) {
      one_block<KM1, DT, BETA, MODE, BI>(bc, tb);
      super_block<KM1, DT, BETA, MODE, BI + 1, NB>(bc, t0);
    }
  }
}

}  // namespace rot

// Wavefronts per workgroup: four, one per SIMD, so that every SIMD of a CU
// receives the same number of frames (the wavefronts share nothing).
constexpr int kRotWaves = 4;

// The frames of wave-table entry 'wave', on one wavefront.
template <int KM1, int DT, int BETA, int MODE>
__device__ __forceinline__ void fwd_rot_wave(const DevCode* __restrict__ codes,
                                             const Item* __restrict__ items,
                                             const int2* __restrict__ waves, int wave,
                                             const void* __restrict__ llr_v,
                                             uint64_t* __restrict__ surv, void* metric,
                                             int32_t* end_out, int32_t* item_end,
                                             typename rot::Ty<DT>::T (*bmt)[32 << BETA],
                                             typename rot::Ty<DT>::T* xpm, int lane) {
  using namespace rot;
  using T = typename Ty<DT>::T;
  using In = typename Ty<DT>::In;
  constexpr int NS = 1 << KM1;
  constexpr int NP = 1 << BETA;
  constexpr int SUPER = 32 * KM1 / gcd_c(32, KM1);  // lcm(32, K-1)
  const int fr = lane / NS, sl = lane % NS;
  // this wave's frames: waves[w] = (first item, count), all of equal length
  const int2 wv = waves[wave];
  const bool valid = fr < wv.y;
  const Item it = items[wv.x + (valid ? fr : 0)];
  const DevCode c = codes[it.code];
  const int S = __builtin_amdgcn_readfirstlane(it.n_stages);  // equal within the wave
  const In* llr = (const In*)llr_v + it.llr_off;
  uint32_t* sv = (uint32_t*)(surv + it.surv_off);

  Frame<KM1, DT, NP, MODE> F;
#pragma unroll
  for (int q = 0; q < KM1; ++q) {
    const int j = rotr(sl, (q + 1) % KM1, KM1);  // state held after a phase-q stage
    const int ie = (j << 1) & (NS - 1);
    const int u = j >> (KM1 - 1);
    // MODE 0: the even previous state's branch into j; MODE 1 (own/partner):
    // its branch on input 0
    F.pat_off[q] = branch_out(c, ie, MODE == 0 ? u : 0);
    uint64_t bm = 0;
    for (int l = 0; l < 64; ++l)
      if ((l >> q) & 1) bm |= 1ull << l;
    F.bmask[q] = bm;
  }
  F.addr_e = (lane & ~32) << 2;
  F.addr_o = (lane | 32) << 2;
  F.addr_p = (lane ^ 32) << 2;
  F.pm = (it.start_known && sl != 0) ? Ty<DT>::neg_unreachable() : (T)0;
  F.acc = 0;
  int64_t offset = 0;
  T* my_bmt = &bmt[fr][0];

  int blk = 0;
  BlockCtx<KM1, DT, BETA, MODE> bc{&F, my_bmt, llr, sv, &offset, &blk, S, sl, lane, valid, {}};
  bc.lr.load(llr, 0, S, sl, valid);
  for (int t0 = 0; t0 < S; t0 += SUPER) super_block<KM1, DT, BETA, MODE, 0, SUPER / 32>(bc, t0);
  // final metrics: lane sl holds state rotr(sl, S mod (K-1))
  const int st = rotr(sl, S % KM1, KM1);
  xpm[fr * NS + st] = F.pm;
  wave_sync();
  if (sl == 0 && valid) {
    int js = it.end_state;
    if (js < 0) {
      js = 0;
      for (int j = 1; j < NS; ++j)
        if (xpm[fr * NS + j] > xpm[fr * NS + js]) js = j;
    }
    item_end[it.slot] = js;
    if (it.frame >= 0) {
      if (end_out) end_out[it.frame] = js;
      if (metric) {
        if constexpr (Ty<DT>::kInt)
          ((int64_t*)metric)[it.frame] = (int64_t)xpm[fr * NS + js] + offset;
        else
          ((float*)metric)[it.frame] = xpm[fr * NS + js];
      }
    }
  }
}

namespace rot {

// ---------------------------------------------------------------------------
// MODE 2: one stage is a short dependent chain, so what a lone wavefront pays
// is its instruction count plus every wait in the chain, and what a full
// device pays is vector instructions.
//
//  - The new metric is v_max of the candidates and the decision the sign bit
//    of their difference, shifted into the lane's word by one v_alignbit: no
//    compare, no lane mask, none of the wait states a mask costs, and the two
//    decision instructions fill the wait states a DPP read needs.
//  - Bits 4 and 5: every lane forms the candidates of its own state's two
//    successors (pm + m and pm - m: the corollary again) and one swap of the
//    two registers hands both candidates of the new state to its lane.
//  - Bits 2, 3: own and partner candidates; in lanes whose own state is the
//    odd one the difference is taken the other way round by a second subtract
//    with a DPP bank mask, so a tie keeps the even state in every lane.
//  - A block's branch metrics are read from LDS one block ahead, each into
//    the register its stage has just consumed, and the table they come from
//    is written one block before that: no stage waits for LDS.
//
// float metrics are the same bits as with a compare and select as long as no
// NaN and no infinity but an unreachable state's -inf occurs (and -0 never
// occurs: sums start from +0).  Soft values below 2^90 in magnitude cannot
// produce any; where others are seen, slow_blocks runs that period again and
// the rest of the frame.
//
// Forward pass alone, K = 7, float, against one compare, select and mask per
// stage: one frame of 1030 stages 35 -> 20 us, 999 of 3001 (a wavefront per
// SIMD) 122 -> 61, 4096 of 8198 (four) 457 -> 367.  There the VALU is the
// bound: 6.2 vector instructions a stage, of which 5 to 7 (by phase) are the
// stage's own.
// ---------------------------------------------------------------------------

// acc = 2 acc + sign bit of t
__device__ __forceinline__ uint32_t push_sign(uint32_t acc, uint32_t t) {
  return __builtin_amdgcn_alignbit(acc, t, 31);
}

// Own/partner stages (Q = 2, 3): the larger candidate, and the difference of
// the even and the odd previous state's: own - partner, taken the other way
// round in the lanes with bit Q set (banks 1, 3 or 2, 3 of each row).  co and
// cp were written before the block; its first two instructions are the wait
// states the DPP read of cp needs.
#define MV_OWN_PARTNER(SUB, MAX, BANKS)                                              \
  asm(SUB " %0, %2, %3\n\t" MAX " %1, %2, %3\n\t" SUB                               \
      "_dpp %0, %3, %2 quad_perm:[0,1,2,3] row_mask:0xf bank_mask:" BANKS            \
      : "=&v"(t), "=&v"(r) : "v"(co), "v"(cp))
template <int Q>
__device__ __forceinline__ float max_and_diff(float co, float cp, uint32_t& diff) {
  float t, r;
  if constexpr (Q == 2)
    MV_OWN_PARTNER("v_sub_f32", "v_max_f32", "0xa");
  else
    MV_OWN_PARTNER("v_sub_f32", "v_max_f32", "0xc");
  diff = __builtin_bit_cast(uint32_t, t);
  return r;
}
template <int Q>
__device__ __forceinline__ int max_and_diff(int co, int cp, uint32_t& diff) {
  int t, r;
  if constexpr (Q == 2)
    MV_OWN_PARTNER("v_sub_u32", "v_max_i32", "0xa");
  else
    MV_OWN_PARTNER("v_sub_u32", "v_max_i32", "0xc");
  diff = (uint32_t)t;
  return r;
}
#undef MV_OWN_PARTNER
__device__ __forceinline__ uint32_t diff_bits(float a, float b) {
  return __builtin_bit_cast(uint32_t, a - b);
}
__device__ __forceinline__ uint32_t diff_bits(int a, int b) { return (uint32_t)(a - b); }
// (v_max directly: the compiler quiets the swaps' results first, two more
// instructions, since it cannot see that they are never signalling NaNs)
__device__ __forceinline__ float vmax(float a, float b) {
  float r;
  asm("v_max_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
__device__ __forceinline__ int vmax(int a, int b) { return a > b ? a : b; }

template <int KM1, int DT, int BETA>
struct Valu {
  using T = typename Ty<DT>::T;
  static constexpr int NS = 1 << KM1, NP = 1 << BETA;
  T pm;
  uint32_t acc;
  T bmv[32];         // branch metrics of the stages ahead
  const T* tp[KM1];  // table row 0 entry of this lane per phase
  T* bmt;
  const typename Ty<DT>::In* llr;
  uint32_t* sv;      // survivor words of the frame, plus this lane
  int64_t offset;
  int S, sl, lane;
  uint64_t bad;      // a soft value for slow_blocks was seen
  // soft values of the blocks ahead, of stages row(k); block b in lr[b % NB]
  static constexpr int NSTG = LlrRegs<KM1, DT, BETA>::NSTG;
  static constexpr int NB0 = KM1 / gcd_c(32, KM1);  // blocks per phase period
  static constexpr int NB = NB0 == 1 ? 2 : NB0;     // and per trip of the main loop
  T lr[NB][NSTG][BETA];
  // block stage of register k: every lane has one (64 lanes: each twice)
  __device__ __forceinline__ int row(int k) const { return NS > 32 ? sl & 31 : sl + k * NS; }
  __device__ __forceinline__ void load(T (&dst)[NSTG][BETA], int tb) {
#pragma unroll
    for (int k = 0; k < NSTG; ++k) {
      const int64_t t = min(tb + row(k), S - 1);  // past the end: not used
#pragma unroll
      for (int b = 0; b < BETA; ++b) dst[k][b] = (T)llr[t * BETA + b];
    }
  }
};

// One stage at phase Q; m: metric of the lane's branch (see table_patterns).
template <int KM1, int DT, int BETA, int Q>
__device__ __forceinline__ void valu_stage(Valu<KM1, DT, BETA>& F, typename Ty<DT>::T m) {
  using T = typename Ty<DT>::T;
  if constexpr (own_partner<Q>) {
    const T cp = partner_fetch_valu<Q, DT>(F.pm) - m;
    const T co = F.pm + m;
    uint32_t t;
    F.pm = max_and_diff<Q>(co, cp, t);
    F.acc = push_sign(F.acc, t);
  } else {
    T ce, co;
    if constexpr (Q < 2) {
      T e, o;
      pair_fetch_valu<Q, DT>(F.pm, e, o);
      ce = e + m;
      co = o - m;
    } else {
      const int c0 = Ty<DT>::bits(F.pm + m), c1 = Ty<DT>::bits(F.pm - m);
      if constexpr (Q == 4) {
        const auto r = __builtin_amdgcn_permlane16_swap(c0, c1, false, false);
        ce = Ty<DT>::from(r[0]);
        co = Ty<DT>::from(r[1]);
      } else {
        const auto r = __builtin_amdgcn_permlane32_swap(c0, c1, false, false);
        ce = Ty<DT>::from(r[0]);
        co = Ty<DT>::from(r[1]);
      }
    }
    F.pm = vmax(ce, co);
    F.acc = push_sign(F.acc, diff_bits(ce, co));
  }
}

// Stages K0 .. 31 of a block whose first stage has phase P0, reading the
// next block's metrics (its first phase is P0 + 32).
template <int KM1, int DT, int BETA, int P0, int K0>
__device__ __forceinline__ void valu_full(Valu<KM1, DT, BETA>& F) {
  if constexpr (K0 < 32) {
    valu_stage<KM1, DT, BETA, (P0 + K0) % KM1>(F, F.bmv[K0]);
    F.bmv[K0] = F.tp[(P0 + 32 + K0) % KM1][K0 * (1 << BETA)];
    valu_full<KM1, DT, BETA, P0, K0 + 1>(F);
  }
}
// Table of Eq. (BM) over all output patterns for the soft values in lr.
template <int KM1, int DT, int BETA>
__device__ __forceinline__ void valu_table(Valu<KM1, DT, BETA>& F,
                                           const typename Ty<DT>::T (&lr)[Valu<KM1, DT, BETA>::NSTG][BETA]) {
  using T = typename Ty<DT>::T;
  constexpr int NP = 1 << BETA;
#pragma unroll
  for (int k = 0; k < F.NSTG; ++k) {
    T* row = F.bmt + F.row(k) * NP;
#pragma unroll
    for (int p = 0; p < NP / 2; ++p) {
      T v = (T)0;
#pragma unroll
      for (int b = 0; b < BETA; ++b) v += ((p >> b) & 1) ? -lr[k][b] : lr[k][b];
      row[p] = v;
      row[NP - 1 - p] = -v;
    }
  }
}

// Note soft values in lr (of any lane) that may bring a NaN or an infinity
// into the metrics.
template <int KM1, int DT, int BETA>
__device__ __forceinline__ void valu_look(Valu<KM1, DT, BETA>& F,
                                          const typename Ty<DT>::T (&lr)[Valu<KM1, DT, BETA>::NSTG][BETA]) {
  if constexpr (!Ty<DT>::kInt) {
    float m = 0.0f;
#pragma unroll
    for (int k = 0; k < F.NSTG; ++k)
#pragma unroll
      for (int b = 0; b < BETA; ++b) m += __builtin_fabsf(lr[k][b]);
    F.bad |= __builtin_amdgcn_ballot_w64(!(m < 0x1p90f));
  }
}

// Range control of integer metrics, once per period (a metric moves by at
// most 512 a stage): back by the metric of state 0, which is in the frame's
// lane 0 there.
template <int KM1, int DT, int BETA>
__device__ __forceinline__ void valu_renorm(Valu<KM1, DT, BETA>& F) {
  if constexpr (Ty<DT>::kInt) {
    constexpr int NS = 1 << KM1;
    int ref;
    if constexpr (NS == 64)
      ref = __builtin_amdgcn_readfirstlane(F.pm);
    else
      ref = __builtin_amdgcn_ds_bpermute((F.lane & ~(NS - 1)) << 2, F.pm);
    F.pm -= ref;
    F.offset += ref;
  }
}

// At the start of block BI (of a trip) at stage tb: the next block's table
// (its metrics' reads follow in program order, and this block's were all
// issued a block ago) and the soft values a trip after it: a lone wavefront
// runs 32 stages in less time than memory takes to answer.
template <int KM1, int DT, int BETA, int BI>
__device__ __forceinline__ void valu_next(Valu<KM1, DT, BETA>& F, int tb) {
  auto& lr = F.lr[(BI + 1) % F.NB];
  valu_look(F, lr);
  valu_table(F, lr);
  F.load(lr, tb + 32 * (F.NB + 1));
  wave_sync();
}

// Blocks BI .. NB-1 of a whole period from t0.
template <int KM1, int DT, int BETA, int BI, int NB>
__device__ __forceinline__ void valu_period(Valu<KM1, DT, BETA>& F, int t0) {
  if constexpr (BI < NB) {
    const int tb = t0 + 32 * BI;
    valu_next<KM1, DT, BETA, BI>(F, tb);
    valu_full<KM1, DT, BETA, (32 * BI) % KM1, 0>(F);
    F.sv[(int64_t)(tb >> 5) << KM1] = F.acc;
    wave_sync();
    valu_period<KM1, DT, BETA, BI + 1, NB>(F, t0);
  }
}

// The last, partial period: n stages from t0.  Leaves after any stage (the
// decisions since the last whole block stay in acc).
template <int KM1, int DT, int BETA, int K, int SUPER>
__device__ __forceinline__ void valu_tail(Valu<KM1, DT, BETA>& F, int t0, int n) {
  if constexpr (K < SUPER - 1) {
    if (K < n) {
      if constexpr (K % 32 == 0) valu_next<KM1, DT, BETA, K / 32>(F, t0 + K);
      valu_stage<KM1, DT, BETA, K % KM1>(F, F.bmv[K % 32]);
      F.bmv[K % 32] = F.tp[(K + 32) % KM1][(K % 32) << BETA];
      if constexpr (K % 32 == 31) {
        F.sv[(int64_t)((t0 + K) >> 5) << KM1] = F.acc;
        wave_sync();
      }
      valu_tail<KM1, DT, BETA, K + 1, SUPER>(F, t0, n);
    }
  }
}

// The frame's stages from t0 on with compare and select as written in Eqs.
// (PM), (SP0): for soft values that bring NaNs or infinities.
template <int KM1, int DT, int BETA, int Q>
__device__ __forceinline__ void slow_stage(Valu<KM1, DT, BETA>& F, const DevCode& c,
                                           const typename Ty<DT>::T* row, int q) {
  using T = typename Ty<DT>::T;
  if constexpr (Q < KM1) {
    if (q != Q) {
      slow_stage<KM1, DT, BETA, Q + 1>(F, c, row, q);
      return;
    }
    const int j = rotr(F.sl, (Q + 1) % KM1, KM1);
    const int ie = (j << 1) & ((1 << KM1) - 1);
    if constexpr (own_partner<Q>) {
      const T m = row[branch_out(c, ie, 0)];
      const T cp = partner_fetch_valu<Q, DT>(F.pm) - m;
      const T co = F.pm + m;
      F.pm = tmax(co, cp);
      const bool odd = (F.lane >> Q) & 1;
      F.acc = 2 * F.acc + (uint32_t)(odd ? co > cp : cp > co);
    } else {
      const T m = row[branch_out(c, ie, j >> (KM1 - 1))];
      T e, o;
      pair_fetch_valu<Q, DT>(F.pm, e, o);
      const T ce = e + m, co = o - m;
      const bool d = co > ce;
      F.pm = d ? co : ce;
      F.acc = 2 * F.acc + (uint32_t)d;
    }
  }
}

template <int KM1, int DT, int BETA>
__device__ __forceinline__ void slow_blocks(Valu<KM1, DT, BETA>& F, const DevCode& c, int t0) {
#pragma unroll 1
  for (int tb = t0; tb < F.S; tb += 32) {
    F.load(F.lr[0], tb);
    wave_sync();
    valu_table(F, F.lr[0]);
    wave_sync();
    const int n = min(32, F.S - tb);
    F.acc = 0;
#pragma unroll 1
    for (int k = 0; k < n; ++k)
      slow_stage<KM1, DT, BETA, 0>(F, c, F.bmt + k * (1 << BETA), (tb + k) % KM1);
    F.sv[(int64_t)(tb >> 5) << KM1] = F.acc << (32 - n);
  }
}

}  // namespace rot

// The frames of wave-table entry 'wave', on one wavefront, MODE 2.
template <int KM1, int DT, int BETA>
__device__ __forceinline__ void fwd_rot_valu_wave(const DevCode* __restrict__ codes,
                                                  const Item* __restrict__ items,
                                                  const int2* __restrict__ waves, int wave,
                                                  const void* __restrict__ llr_v,
                                                  uint64_t* __restrict__ surv, void* metric,
                                                  int32_t* end_out, int32_t* item_end,
                                                  typename rot::Ty<DT>::T (*bmt)[32 << BETA],
                                                  typename rot::Ty<DT>::T* xpm, int lane) {
  using namespace rot;
  using T = typename Ty<DT>::T;
  constexpr int NS = 1 << KM1;
  constexpr int SUPER = 32 * Valu<KM1, DT, BETA>::NB;  // whole phase periods
  const int fr = lane / NS, sl = lane % NS;
  const int2 wv = waves[wave];
  // lanes beyond the entry's frames repeat its first frame (same inputs, same
  // stores)
  const bool valid = fr < wv.y;
  const Item it = items[wv.x + (valid ? fr : 0)];
  const DevCode c = codes[it.code];
  Valu<KM1, DT, BETA> F;
  F.S = __builtin_amdgcn_readfirstlane(it.n_stages);  // equal within the wave
  F.sl = sl;
  F.lane = lane;
  F.bad = 0;
  F.llr = (const typename Ty<DT>::In*)llr_v + it.llr_off;
  F.sv = (uint32_t*)(surv + it.surv_off) + sl;
  F.bmt = &bmt[fr][0];
  F.offset = 0;
  F.acc = 0;
  F.pm = (it.start_known && sl != 0) ? Ty<DT>::neg_unreachable() : (T)0;
#pragma unroll
  for (int q = 0; q < KM1; ++q) {
    // bits 0, 1: the even previous state's branch into the new state; bits
    // 2, 3: that state's branch on input 0; bits 4, 5: the branch on input 0
    // of the state the lane holds before the stage
    const int j = rotr(sl, (q + 1) % KM1, KM1);
    const int ie = (j << 1) & (NS - 1);
    const int own = rotr(sl, q, KM1);
    F.tp[q] = F.bmt + (q < 2 ? branch_out(c, ie, j >> (KM1 - 1))
                             : q < 4 ? branch_out(c, ie, 0) : branch_out(c, own, 0));
  }
  if (F.S > 0) {
#pragma unroll
    for (int b = 0; b < F.NB; ++b) F.load(F.lr[b], 32 * b);
    valu_look(F, F.lr[0]);
    valu_table(F, F.lr[0]);
    F.load(F.lr[0], 32 * F.NB);
    wave_sync();
#pragma unroll
    for (int k = 0; k < 32; ++k) F.bmv[k] = F.tp[k % KM1][k * (1 << BETA)];
    int t0 = 0;
    T pm0 = F.pm;  // metrics entering the period from t0
    // Only where wavefronts share SIMDs, and for float32: 4096 frames of 8198
    // stages, decode, 416 -> 408 us; float16 took 376 against 369 with it.
    const int slot = DT == 0 && gridDim.x > kComputeUnits ? wave_slot() : -1;
    for (; t0 + SUPER <= F.S && F.bad == 0; t0 += SUPER) {
      pm0 = F.pm;
      valu_period<KM1, DT, BETA, 0, SUPER / 32>(F, t0);
      valu_renorm(F);
      if (slot >= 0) fair_share(slot, t0 / SUPER);
    }
    if (F.bad != 0) {
      t0 = max(t0 - SUPER, 0);
    } else {
      pm0 = F.pm;
      valu_tail<KM1, DT, BETA, 0, SUPER>(F, t0, F.S - t0);
      const int rem = F.S & 31;
      if (rem) F.sv[(int64_t)(F.S >> 5) << KM1] = F.acc << (32 - rem);
    }
    if constexpr (!Ty<DT>::kInt) {
      if (F.bad != 0) {
        // the period in which they were seen, again
        F.pm = pm0;
        slow_blocks(F, c, t0);
      }
    }
  }
  // final metrics: lane sl holds state rotr(sl, S mod (K-1)); the best state,
  // ties to the lowest index
  const int st = rotr(sl, F.S % KM1, KM1);
  xpm[fr * NS + st] = F.pm;
  wave_sync();
  if (sl == 0 && valid) {
    int js = it.end_state;
    if (js < 0) {
      js = 0;
      for (int j = 1; j < NS; ++j)
        if (xpm[fr * NS + j] > xpm[fr * NS + js]) js = j;
    }
    item_end[it.slot] = js;
    if (it.frame >= 0) {
      if (end_out) end_out[it.frame] = js;
      if (metric) {
        if constexpr (Ty<DT>::kInt)
          ((int64_t*)metric)[it.frame] = (int64_t)xpm[fr * NS + js] + F.offset;
        else
          ((float*)metric)[it.frame] = xpm[fr * NS + js];
      }
    }
  }
}

// One wavefront per wave-table entry, or (counter != nullptr) a persistent
// grid whose wavefronts take entries in table order (longest frames first)
// from a device counter that starts at zero, until the table is exhausted.
//
// Wavefronts per SIMD the registers are held to, MODE 2: five, but four for
// rate 1/4 with K = 6, 7, whose periods would reload spilled registers (forward
// pass, 10000 wavefronts of 517 stages, five / four per SIMD: K = 6 rate 1/4
// float32 94 / 75 us, float16 130 / 76; K = 7 rate 1/4 float16 77 / 72).  The
// other codes spill around their periods only, which a full device hides (4096
// frames of 8192 bits, decode, five / four: K = 4 rate 1/2 float32 183 / 196,
// K = 5 rate 1/4 int8 271 / 291, K = 5 rate 1/2 float32 177 / 184).
constexpr int rot_occupancy(int KM1, int BETA) { return KM1 >= 5 && BETA == 4 ? 4 : 5; }
template <int KM1, int DT, int BETA, int MODE>
__global__ __launch_bounds__(64 * kRotWaves, MODE == 2 ? rot_occupancy(KM1, BETA) : 1) void k_fwd_rot(const DevCode* __restrict__ codes,
                                                const Item* __restrict__ items,
                                                const int2* __restrict__ waves, int n_waves,
                                                const void* __restrict__ llr_v,
                                                uint64_t* __restrict__ surv, void* metric,
                                                int32_t* end_out, int32_t* item_end,
                                                int32_t* counter) {
  using T = typename rot::Ty<DT>::T;
  constexpr int FPW = 64 >> KM1;
  __shared__ T bmt_all[kRotWaves][FPW][32 << BETA];
  __shared__ T xpm_all[kRotWaves][64];
  const int wid = threadIdx.x >> 6;
  const int lane = threadIdx.x & 63;
  if (counter == nullptr) {
    const int wave = blockIdx.x * kRotWaves + wid;
    if (wave >= n_waves) return;  // no workgroup barriers: safe to leave
    if constexpr (MODE == 2)
      fwd_rot_valu_wave<KM1, DT, BETA>(codes, items, waves, wave, llr_v, surv, metric, end_out,
                                       item_end, bmt_all[wid], xpm_all[wid], lane);
    else
      fwd_rot_wave<KM1, DT, BETA, MODE>(codes, items, waves, wave, llr_v, surv, metric, end_out,
                                         item_end, bmt_all[wid], xpm_all[wid], lane);
    return;
  }
  for (;;) {
    int w = 0;
    if (lane == 0) w = atomicAdd(counter, 1);
    w = __builtin_amdgcn_readfirstlane(w);
    if (w >= n_waves) break;
    if constexpr (MODE == 2)
      fwd_rot_valu_wave<KM1, DT, BETA>(codes, items, waves, w, llr_v, surv, metric, end_out,
                                       item_end, bmt_all[wid], xpm_all[wid], lane);
    else
      fwd_rot_wave<KM1, DT, BETA, MODE>(codes, items, waves, w, llr_v, surv, metric, end_out,
                                         item_end, bmt_all[wid], xpm_all[wid], lane);
  }
}

// Launch one instantiation: a workgroup of kRotWaves per table entries, or
// the resident grid for a persistent launch.
template <typename Kernel>
hipError_t rot_go(Kernel kernel, const DevCode* codes, const Item* items, const int2* waves,
                  int n_waves, const void* llr, uint64_t* surv, void* metric, int32_t* end_out,
                  int32_t* item_end, int32_t* counter, int grid_limit, hipStream_t st) {
  const int threads = 64 * kRotWaves;
  int nb = (n_waves + kRotWaves - 1) / kRotWaves;
  if (counter) {
    const int lim = grid_limit > 0 ? grid_limit : resident_workgroups(kernel, threads);
    if (lim > 0 && nb > lim) nb = lim;
  }
  hipLaunchKernelGGL(kernel, dim3(nb), dim3(threads), 0, st, codes, items, waves, n_waves, llr,
                     surv, metric, end_out, item_end, counter);
  return hipGetLastError();
}

#define MV_ROT_ARGS                                                                            \
  int K, int beta, const DevCode *codes, const Item *items, const int2 *waves, int n_waves,    \
      const void *llr, uint64_t *surv, void *metric, int32_t *end_out, int32_t *item_end,      \
      int32_t *counter, int grid_limit, hipStream_t st
#define MV_ROT_PASS                                                                            \
  codes, items, waves, n_waves, llr, surv, metric, end_out, item_end, counter, grid_limit, st

// One type and mode, all codes with K <= 7.
template <int DT, int MODE>
hipError_t rot_launch(MV_ROT_ARGS) {
  switch (K * 8 + beta) {
#define MV_ROT_K(KM1)                                                        \
  case (KM1 + 1) * 8 + 2: return rot_go(k_fwd_rot<KM1, DT, 2, MODE>, MV_ROT_PASS); \
  case (KM1 + 1) * 8 + 3: return rot_go(k_fwd_rot<KM1, DT, 3, MODE>, MV_ROT_PASS); \
  case (KM1 + 1) * 8 + 4: return rot_go(k_fwd_rot<KM1, DT, 4, MODE>, MV_ROT_PASS)
    MV_ROT_K(2);
    MV_ROT_K(3);
    MV_ROT_K(4);
    MV_ROT_K(5);
    MV_ROT_K(6);
#undef MV_ROT_K
    default: return hipErrorInvalidValue;
  }
}

// The default mode, one source file per soft-value type (they compile side
// by side).
hipError_t launch_rot_f32(MV_ROT_ARGS);
hipError_t launch_rot_i8(MV_ROT_ARGS);
hipError_t launch_rot_f16(MV_ROT_ARGS);

}  // namespace mivit

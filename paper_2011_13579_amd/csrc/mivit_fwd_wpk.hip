// Forward procedure for K = 8 and 9, int8 soft values, beta = 2 or 3: two
// states of a frame packed in the 16-bit halves of every register, two
// radix-2 stages per iteration, radix-4 survivors.
//
// Metrics.  A half holds 4 (PM + offset) + 3 + h, h the history of the current
// iteration: a stage's even candidate adds t = 4 m + g and its odd candidate
// subtracts the same t (by the corollary of §IV the two branches into a state
// have opposite metrics m), g = 1 for the first stage of an iteration and 2
// for the second.  All path metrics of a frame at one time have the same
// parity (every branch metric of a stage has the parity of the sum of its
// soft values), so different metrics are 8 apart and a history never decides
// between them; equal ones go to the even previous state (R1).  After both
// stages the parity is taken back (at most one unit per stage, a table word),
// which leaves 3 + h = 6 - 2y in bits 1 and 2, y the radix-4 digit; they are
// collected and cleared.  t is the low half's value plus 65536 times the
// high half's, both signed; every half of the true sums lies in [0, 65535],
// so no carry or borrow is lost.  Per register and iteration that is six
// instructions for the stages and four for parity and digits, where a stage
// by itself (two biased additions, maximum, clear and collect the tag) took
// six.
//
// Range control.  The metrics of a frame's states never differ by more than
// W = 256 beta (K-1), and the best one falls by at most the parities.  State
// 0 is brought to C = W + 128 beta + 32 every 8 stages: every metric and
// candidate stays in [0, 2 W + 9 x 128 beta + 64], 14 bits for beta = 3.  From
// a known start every state is reached before the first range control.
//
// Positions.  At time t the state s has the rotated index r = rotl_n(s, t mod
// n), n = K-1, so that stage t pairs the indices that differ in bit q = t mod
// n.  Index bits 0 to 5 name the lane (lane bits 0 and 1 xored with bit 2, as
// in the packed K = 7 kernel: the partners for q < 4 are one DPP pattern
// each), for q = 4, 5 the candidates a lane forms for its own state's two
// successors are swapped by v_permlane16/32_swap; K = 9: bit 6 names the
// register, where nothing moves; the top bit names the half.
//
// Branch metrics.  Per stage 2^(beta+1) words: t for every pattern of the low
// half's state (the high half's differs by a pattern that depends on the
// phase only), and -t for lanes whose own previous state is the odd one.  A
// block of tables is 32 stages (K = 8: 28, whole phase periods), a lane fills
// half a row of the next block; two blocks rotate in LDS.
//
// Odd stage counts: stage 0 is evaluated in closed form and the rest counts
// from it; the traceback emits its bit from the state at time 1.
//
// Survivors: per 8 stages 2^n bytes, index r at byte (r mod 64) 2^(n-6) +
// (r >> 6), so that a lane's bytes are one word; the digit y of iteration i of
// the group in bits 6 - 2i and up.
//
// What bounds it: vector issue, 12.6 instructions per stage for K = 9 (15 and
// LDS swizzles with one stage at a time), and with one or two wavefronts per
// SIMD the latency of each stage's chain.  Measured, K = 9 rate 1/3, against
// that kernel (which left repairs to two more launches): 512 frames of 4000
// bits, forward 125 -> 82 us, with the check 141 -> 86, decode 153 -> 103; 4096
// of 2000 bits, decode 308 -> 272, one of 4096 (in eight parts) 52; K = 8 rate
// 1/2, 4096 of 2000 bits 173 -> 162.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "mivit_device.h"
#include "mivit_fwd_wide.h"

namespace mivit {

namespace wpk {

using wide::branch_out;
using wide::rotl;
using wide::rotr;
using wide::wave_sync;

constexpr uint32_t kBoth = 0x10001u;
constexpr uint32_t kTag = 6 * kBoth;
constexpr int kWaves = 4;  // wavefronts per workgroup (they share nothing)

typedef unsigned short us2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pk_max(uint32_t a, uint32_t b) {
  return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(us2, a),
                                                                __builtin_bit_cast(us2, b)));
}

// lane <-> low six index bits (its own inverse)
__device__ __forceinline__ int index_of(int p) { return p ^ ((p & 4) ? 3 : 0); }

template <int Q>
__device__ __forceinline__ uint32_t partner(uint32_t x) {
  constexpr int ctrl = Q == 0 ? 0xB1 : Q == 1 ? 0x4E : Q == 2 ? 0x141 : 0x128;
  return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, ctrl, 0xF, 0xF, true);
}

template <int N, int BETA>
struct Fwd {
  static constexpr int NS = 1 << N, V = NS / 128, NP = 1 << BETA;
  static constexpr int kRows = N == 8 ? 32 : 28;  // stages per table block
  static constexpr int kBufs = 2;
  static constexpr int kTrip = wpk_period(N);     // whole phase periods and groups
  static constexpr int kRow = 2 * NP + 4;         // words per row: t, -t, parity, padding
  static constexpr int kBuf = kRows * kRow;
  static constexpr int kAhead = 4;                // stages an entry is read ahead
  static constexpr int kRen = 8;                  // stages between range controls
  static constexpr int kOut = 128 * BETA;         // largest branch metric
  static constexpr int kSpread = 2 * N * kOut;
  static constexpr int kC = kSpread + kOut + 32;
  // a known start: state 0 above what the others can make up in N stages
  // (and stage 0 of an odd count), and these above 0 meanwhile
  static constexpr int kUnreach = 8 * kOut + 32;
  static constexpr int kKnown = kUnreach + 17 * kOut + 32;
  static_assert(4 * (kC + kSpread + kRen * kOut) + 7 < 65536, "16-bit range");
  static_assert(4 * (kKnown + 9 * kOut) + 7 < 65536, "16-bit range from a known start");
  static_assert(kTrip % 16 == 0 && kTrip % N == 0 && kTrip % (kBufs * kRows) == 0, "trip");
  static_assert(kRows % N == 0 && kRows % 2 == 0, "a row's phase does not depend on the block");
  const uint32_t* tp[N][V];   // table entry (row 0, buffer 0) per phase and register
  const uint32_t* tp1[2][V];  // entry of the candidate for input 1, bits 4 and 5
  const uint32_t* pp;         // parity word
  uint32_t* trow;             // table words this lane fills (buffer 0)
  uint32_t* prow;
  uint32_t g;                 // g of this lane's row in both halves, with its sign
  int32_t k[BETA];            // soft value -> both halves, with their signs
  const int8_t* l0;           // soft values of stage 0
  int w[kBufs][BETA];         // those of this lane's row, blocks ahead
  uint32_t pm[V];
  uint32_t q[kAhead][V], q1[kAhead][V];  // entries of the stages ahead
  uint32_t qp[2];             // parity words of the iterations ahead
  uint32_t strip, three;      // ~7 and 3 in both halves, in registers: one v_and_or
  uint32_t acc[V];            // digits of the current group
  uint8_t* sv;                // survivor bytes, plus this lane's place
  int row, last, end;         // row; last stage that can be loaded; stages that count
  uint32_t par, par_ahead;    // parities of this lane's rows; those of the block ahead
  int off;                    // subtracted by range control in the current trips
  int64_t sum;                // and in those before
};

template <int N, int BETA>
__device__ __forceinline__ void load(Fwd<N, BETA>& F, int b, int stage) {
  const int8_t* p = F.l0 + (int64_t)BETA * min(stage + F.row, F.last);
#pragma unroll
  for (int i = 0; i < BETA; ++i) F.w[b][i] = p[i];
}

// This lane's half row from its soft values (stage: the block's first), into
// buffer `buf`: lanes below 32 the words t, the others -t.
template <int N, int BETA>
__device__ __forceinline__ void table(Fwd<N, BETA>& F, int b, int buf, int stage, int lane) {
  using W = Fwd<N, BETA>;
  uint32_t L[BETA], s[W::NP];
#pragma unroll
  for (int i = 0; i < BETA; ++i) L[i] = (uint32_t)__mul24(F.w[b][i], F.k[i]);
  const uint32_t hi = BETA == 3 ? L[2] + L[1] : L[1], lo = BETA == 3 ? L[2] - L[1] : 0u;
  s[0] = hi + L[0];
  s[1] = hi - L[0];
  if constexpr (BETA == 3) {
    s[2] = lo + L[0];
    s[3] = lo - L[0];
  }
#pragma unroll
  for (int x = 0; x < W::NP / 2; ++x) {
    const uint32_t e = (s[x] << 2) + F.g;
    s[x] = e;
    s[W::NP - 1 - x] = 2 * F.g - e;
  }
  uint4* dst = (uint4*)(F.trow + buf * W::kBuf);
#pragma unroll
  for (int x = 0; x < W::NP; x += 4) dst[x / 4] = make_uint4(s[x], s[x + 1], s[x + 2], s[x + 3]);
  uint32_t p = (uint32_t)(F.w[b][0] ^ F.w[b][1]);
  if constexpr (BETA == 3) p ^= (uint32_t)F.w[b][2];
  p &= 1u;
  const uint32_t both = p + partner<0>(p);  // of the iteration
  F.prow[buf * W::kBuf] = both * (4 * kBoth);
  F.par_ahead = (lane < W::kRows && stage + F.row < F.end) ? p : 0u;
  F.par += F.par_ahead;
}

// Entries of stage K of a trip (K may run into the next trip).
template <int N, int BETA, int K>
__device__ __forceinline__ void fetch(Fwd<N, BETA>& F) {
  using W = Fwd<N, BETA>;
  constexpr int q = K % N, o = (K / W::kRows % W::kBufs) * W::kBuf + (K % W::kRows) * W::kRow;
#pragma unroll
  for (int v = 0; v < W::V; ++v) {
    F.q[K % W::kAhead][v] = F.tp[q][v][o];
    if constexpr (q == 4 || q == 5) F.q1[K % W::kAhead][v] = F.tp1[q - 4][v][o];
  }
  if constexpr (K & 1) F.qp[(K >> 1) & 1] = F.pp[o];
}

template <int N, int BETA, int K>
__device__ __forceinline__ void first(Fwd<N, BETA>& F) {
  if constexpr (K < Fwd<N, BETA>::kAhead) {
    fetch<N, BETA, K>(F);
    first<N, BETA, K + 1>(F);
  }
}

template <int N, int BETA, int K>
__device__ __forceinline__ void stage(Fwd<N, BETA>& F) {
  using W = Fwd<N, BETA>;
  constexpr int Q = K % N, V = W::V, A = K % W::kAhead;
  uint32_t c[V], e[V];
#pragma unroll
  for (int v = 0; v < V; ++v) {
    const uint32_t t = F.q[A][v], x = F.pm[v];
    if constexpr (Q < 4) {
      c[v] = x + t;
      e[v] = partner<Q>(x) - t;
    } else if constexpr (Q < 6) {
      const uint32_t c0 = x + t, c1 = x + F.q1[A][v];
      if constexpr (Q == 4) {
        const auto s = __builtin_amdgcn_permlane16_swap(c0, c1, false, false);
        c[v] = s[0];
        e[v] = s[1];
      } else {
        const auto s = __builtin_amdgcn_permlane32_swap(c0, c1, false, false);
        c[v] = s[0];
        e[v] = s[1];
      }
    } else if constexpr (Q < N - 1) {  // the register bit
      c[v] = F.pm[v & ~1] + t;
      e[v] = F.pm[v | 1] - t;
    } else {  // the half bit
      c[v] = __builtin_amdgcn_perm(x, x, 0x01000100u) + t;
      e[v] = __builtin_amdgcn_perm(x, x, 0x03020302u) - t;
    }
  }
#pragma unroll
  for (int v = 0; v < V; ++v) F.pm[v] = pk_max(c[v], e[v]);
}

// The digits of a group, this lane's bytes; short: iterations it lacks.
template <int N, int BETA>
__device__ __forceinline__ void store(Fwd<N, BETA>& F, int group, int lacks) {
  using W = Fwd<N, BETA>;
  uint32_t a[W::V];
#pragma unroll
  for (int v = 0; v < W::V; ++v) a[v] = (F.acc[v] << (2 * lacks)) >> 1;
  uint8_t* dst = F.sv + (int64_t)group * W::NS;
  if constexpr (W::V == 2)
    *(uint32_t*)dst = ~__builtin_amdgcn_perm(a[1], a[0], 0x06020400u);
  else
    *(uint16_t*)dst = (uint16_t)~__builtin_amdgcn_perm(a[0], a[0], 0x0C0C0200u);
}

// The iteration that ends with stage K of a trip is complete: take back its
// parity, collect its digits and clear them; every kRen stages bring state 0
// (lane 0, register 0, low half) to kC.
template <int N, int BETA, bool STORE, int K>
__device__ __forceinline__ void iteration_end(Fwd<N, BETA>& F, uint32_t par, int t0) {
  using W = Fwd<N, BETA>;
  constexpr int k = (K / 2) & 3;  // iteration of the group
#pragma unroll
  for (int v = 0; v < W::V; ++v) {
    const uint32_t x = F.pm[v] - par;
    F.pm[v] = (x & F.strip) | F.three;
    if constexpr (STORE) F.acc[v] = k == 0 ? x & kTag : (F.acc[v] << 2) | (x & kTag);
  }
  if constexpr ((K + 1) % W::kRen == 0) {
    const int d = (int)(__builtin_amdgcn_readfirstlane(F.pm[0]) & 0xFFFFu) - (4 * W::kC + 3);
#pragma unroll
    for (int v = 0; v < W::V; ++v) F.pm[v] -= (uint32_t)d * kBoth;
    F.off += d;
  }
  if constexpr (STORE && k == 3) store(F, (t0 + K) >> 3, 0);
}

template <int N, int BETA, bool STORE, int K>
__device__ __forceinline__ void step(Fwd<N, BETA>& F, int t0, int lane) {
  using W = Fwd<N, BETA>;
  if constexpr (K % W::kRows == 0) {
    constexpr int b = (K / W::kRows + 1) % W::kBufs;  // the next block
    table(F, b, b, t0 + K + W::kRows, lane);
    load(F, b, t0 + K + (W::kBufs + 1) * W::kRows);
    wave_sync();
  }
  const uint32_t par = F.qp[(K >> 1) & 1];
  stage<N, BETA, K>(F);
  fetch<N, BETA, K + W::kAhead>(F);
  if constexpr (K & 1) iteration_end<N, BETA, STORE, K>(F, par, t0);
  if constexpr (K & 1) __builtin_amdgcn_sched_barrier(0);  // reads ahead of their stages
}

template <int N, int BETA, bool STORE, int K>
__device__ __forceinline__ void trip(Fwd<N, BETA>& F, int t0, int lane) {
  if constexpr (K < Fwd<N, BETA>::kTrip) {
    step<N, BETA, STORE, K>(F, t0, lane);
    trip<N, BETA, STORE, K + 1>(F, t0, lane);
  }
}

// The last, partial trip: n (even) stages from t0.
template <int N, int BETA, int K>
__device__ __forceinline__ void tail(Fwd<N, BETA>& F, int t0, int n, int lane) {
  if constexpr (K < Fwd<N, BETA>::kTrip - 2) {
    step<N, BETA, true, K>(F, t0, lane);
    step<N, BETA, true, K + 1>(F, t0, lane);
    if (K + 2 == n) {
      constexpr int k = (K / 2) & 3;
      if constexpr (k != 3) store(F, (t0 + K) >> 3, 3 - k);
    } else {
      tail<N, BETA, K + 2>(F, t0, n, lane);
    }
  }
}

// One wavefront runs the stages of one unit: a whole item, or one part of an
// item split in time (kind 0), or a repair (kind 1).  A part after the first
// warms up from all-zero metrics without storing; a part before the last
// leaves its end metrics in a boundary record; the last part reports the end
// state and its own metric, which the check completes.
template <int N, int BETA>
__device__ __forceinline__ void unit(const DevCode& c, const Item& it, const SplitUnit U, int kind,
                                     WideBound* bounds, int64_t* last_m, const int64_t* rep_m0,
                                     const int8_t* __restrict__ llr, uint64_t* __restrict__ surv,
                                     int64_t* metric, int32_t* end_out, int32_t* item_end,
                                     uint32_t* tbl, int lane) {
  using W = Fwd<N, BETA>;
  constexpr int NS = W::NS, V = W::V, NP = W::NP;
  const int S = __builtin_amdgcn_readfirstlane(it.n_stages);
  const int lead = S & 1;
  const int t_b = U.it_begin, t_e = U.it_end & ~1, t_s = U.it_begin - U.warm;
  const bool first_part = kind == 0 && U.part == 0;
  const bool split = U.n_parts > 1;

  W F;
  F.row = (lane & 31) < W::kRows ? lane & 31 : (lane & 31) - 4;
  F.last = S - lead - 1;
  F.end = t_e;
  F.l0 = llr + it.llr_off + lead * BETA;
  F.trow = tbl + F.row * W::kRow + (lane < 32 ? 0 : NP);
  F.prow = tbl + F.row * W::kRow + 2 * NP;
  F.pp = tbl + 2 * NP;
  F.sv = (uint8_t*)(surv + it.surv_off) + 2 * V * index_of(lane);
  F.par = F.par_ahead = 0;
  // register copies the compiler does not fold back into two literals
  asm volatile("s_mov_b32 %0, %1" : "=s"(F.strip) : "n"(0xFFF8FFF8u));
  asm volatile("v_mov_b32 %0, %1" : "=v"(F.three) : "n"(3 * kBoth));
  F.off = 0;
  F.sum = 0;
  {
    const int sgn = lane < 32 ? 1 : -1;
    F.g = (uint32_t)(sgn * ((F.row & 1) ? 2 : 1)) * kBoth;
    // the register bit of (j << 1) that the half bit of the index flips at
    // this row's phase: the outputs it reaches differ between the halves
    const int b = (2 * N - 2 - F.row % N) % N + 1;
#pragma unroll
    for (int i = 0; i < BETA; ++i)
      F.k[i] = sgn * (((c.gen[i] >> b) & 1u) ? 1 - 65536 : 1 + 65536);
  }
#pragma unroll
  for (int q = 0; q < N; ++q) {
#pragma unroll
    for (int v = 0; v < V; ++v) {
      const int x = index_of(lane) + 64 * v;  // the low half's index
      const bool odd = (x >> q) & 1;          // the lane's own previous state is the odd one
      if (q == 4 || q == 5) {
        const int p0 = branch_out(c, rotr(x, q, N), 0);
        F.tp[q][v] = tbl + (odd ? NP + ((NP - 1) ^ p0) : p0);
        F.tp1[q == 4 ? 0 : 1][v] = tbl + (odd ? NP + p0 : (NP - 1) ^ p0);
      } else {
        const int j = rotr(x, (q + 1) % N, N);
        const int pe = branch_out(c, (j << 1) & (NS - 1), j >> (N - 1));
        F.tp[q][v] = tbl + (q < 4 && odd ? NP + pe : pe);
      }
    }
  }

  // metrics entering stage t_s: at a whole number of phase periods, so the
  // rotated index is the state
  int c_init = W::kC, p_lead = 0;
  if (first_part) {
    int l[BETA];
#pragma unroll
    for (int i = 0; i < BETA; ++i) {
      l[i] = lead ? (int)llr[it.llr_off + i] : 0;
      p_lead ^= l[i] & 1;
    }
    const bool known = it.start_known != 0;
    if (known) c_init = W::kKnown;
#pragma unroll
    for (int v = 0; v < V; ++v) {
      uint32_t half[2];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int j = index_of(lane) + 64 * (v + V * h);
        int pm = 0;
        bool reach = !known || j == 0;
        if (lead) {
          const int i0 = (j << 1) & (NS - 1);
          const int w = branch_out(c, i0, j >> (N - 1));
          int bm = 0;
#pragma unroll
          for (int i = 0; i < BETA; ++i) bm += ((w >> i) & 1) ? -l[i] : l[i];
          reach = !known || i0 == 0;
          pm = (known ? bm : (bm < 0 ? -bm : bm)) - p_lead;  // unknown start: max(bm, -bm)
        }
        half[h] = 4u * (uint32_t)(reach ? c_init + pm : W::kUnreach) + 3u;
      }
      F.pm[v] = half[0] | (half[1] << 16);
    }
  } else if (kind == 0) {
#pragma unroll
    for (int v = 0; v < V; ++v) F.pm[v] = (uint32_t)(4 * W::kC + 3) * kBoth;  // unknown start
  } else {
    const WideBound& B = bounds[U.bnd + U.part - 1];
#pragma unroll
    for (int v = 0; v < V; ++v) F.pm[v] = (uint32_t)B.v_end[64 * v + lane];  // repair
  }
  // what has been taken from the metrics since t_s (drop: parities of a block
  // not run yet)
  auto taken = [&](uint32_t drop) -> int64_t {
    int p = (int)(F.par - drop);
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) p += __shfl_xor(p, o);
    return (F.sum + F.off) / 4 + p + p_lead;
  };
  if (t_e > t_s) {
#pragma unroll
    for (int b = 0; b < W::kBufs; ++b) load(F, b, t_s + W::kRows * b);
    table(F, 0, 0, t_s, lane);
    load(F, 0, t_s + W::kBufs * W::kRows);
    wave_sync();
    first<N, BETA, 0>(F);
    // (only where wavefronts share SIMDs)
    const int slot = gridDim.x > kComputeUnits ? wave_slot() : -1;
    int t0 = t_s;
    for (; t0 < t_b; t0 += W::kTrip) trip<N, BETA, false, 0>(F, t0, lane);  // warm-up
    if (kind == 0 && U.part > 0) {
      WideBound& B = bounds[U.bnd + U.part - 1];
#pragma unroll
      for (int v = 0; v < V; ++v) B.v_start[64 * v + lane] = (int32_t)F.pm[v];
      const int64_t m = W::kC - c_init + taken(F.par_ahead);
      if (lane == 0) B.m_start = m;
    }
    for (; t0 + W::kTrip <= t_e; t0 += W::kTrip) {
      if (slot >= 0) fair_share(slot, (t0 - t_s) / W::kTrip);
      trip<N, BETA, true, 0>(F, t0, lane);
      F.sum += F.off;
      F.off = 0;
    }
    if (t0 < t_e) tail<N, BETA, 0>(F, t0, t_e - t0, lane);
  }
  const int64_t shift = taken(0) - c_init;
  if (kind == 0 && split && U.part < U.n_parts - 1) {
    WideBound& B = bounds[U.bnd + U.part];
#pragma unroll
    for (int v = 0; v < V; ++v) B.v_end[64 * v + lane] = (int32_t)F.pm[v];
    if (lane == 0) B.m_end = W::kC + shift;
    return;
  }

  // final metrics: index r holds state rotr(r, t_e mod n); the best with ties
  // to the lowest index, and the wanted state's
  const int rot = t_e % N;
  uint32_t key = 0;
#pragma unroll
  for (int r = 0; r < 2 * V; ++r) {
    const uint32_t val = (F.pm[r % V] >> (16 * (r / V))) & 0xFFFFu;
    const uint32_t k = (val << 8) | (uint32_t)(255 - rotr(index_of(lane) + 64 * r, rot, N));
    key = k > key ? k : key;
  }
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t other = (uint32_t)__shfl_xor((int)key, o);
    key = other > key ? other : key;
  }
  const bool fixed = it.end_state >= 0;
  const int js = fixed ? it.end_state : 255 - (int)(key & 255);
  const int x = rotl(js & (NS - 1), rot, N);
  uint32_t vfix = 0;
#pragma unroll
  for (int r = 0; r < 2 * V; ++r) {
    const uint32_t y =
        ((uint32_t)__shfl((int)F.pm[r % V], index_of(x & 63)) >> (16 * (r / V))) & 0xFFFFu;
    vfix = (x >> 6) == r ? y : vfix;
  }
  const int64_t local = (int64_t)((fixed ? vfix : key >> 8) >> 2) + shift;
  if (lane == 0) {
    item_end[it.slot] = js;
    if (it.frame >= 0 && end_out) end_out[it.frame] = js;
    if (kind == 0 && split)
      last_m[it.slot] = local;  // completed by the check
    else if (it.frame >= 0 && metric)
      metric[it.frame] = local + (kind == 1 ? rep_m0[it.slot] : 0);
  }
}

}  // namespace wpk

template <int N, int BETA>
__global__ __launch_bounds__(64 * wpk::kWaves, 4) void k_fwd_wpk(
    const DevCode* __restrict__ codes, const Item* __restrict__ items,
    const SplitUnit* __restrict__ units, int n_units, WideBound* bounds, int64_t* last_m,
    const int8_t* __restrict__ llr, uint64_t* __restrict__ surv, int64_t* metric,
    int32_t* end_out, int32_t* item_end) {
  using W = wpk::Fwd<N, BETA>;
  __shared__ __align__(16) uint32_t tbl_all[wpk::kWaves][W::kBufs * W::kBuf];
  const int wid = threadIdx.x >> 6;
  const int u = __builtin_amdgcn_readfirstlane(blockIdx.x * wpk::kWaves + wid);
  if (u >= n_units) return;  // no workgroup barriers: safe to leave
  const SplitUnit U = units[u];
  const Item it = items[U.first];
  const DevCode c = codes[it.code];
  wpk::unit<N, BETA>(c, it, U, 0, bounds, last_m, nullptr, llr, surv, metric, end_out, item_end,
                     tbl_all[wid], threadIdx.x & 63);
}

// The check after a split forward pass, one wavefront per split item (its
// part-0 unit): boundary k is exact when part k's metrics at its end equal
// part k+1's after its warm-up (both are range-controlled to state 0 there);
// then the metric is the last part's plus the accumulated constants.  Every
// boundary is loaded at once.  An item with an inexact boundary is run again
// from there, from the true metrics, by the same wavefront.
template <int N, int BETA>
__global__ __launch_bounds__(64 * wpk::kWaves, 4) void k_wpk_check(
    const DevCode* __restrict__ codes, const Item* __restrict__ items,
    const SplitUnit* __restrict__ split, int n_split, const SplitUnit* __restrict__ units,
    WideBound* bounds,
    const int64_t* __restrict__ last_m, int64_t* rep_m0, const int8_t* __restrict__ llr,
    uint64_t* __restrict__ surv, int64_t* metric, int32_t* end_out, int32_t* item_end) {
  using W = wpk::Fwd<N, BETA>;
  __shared__ __align__(16) uint32_t tbl_all[wpk::kWaves][W::kBufs * W::kBuf];
  const int wid = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int e = __builtin_amdgcn_readfirstlane(blockIdx.x * wpk::kWaves + wid);
  if (e >= n_split) return;  // no workgroup barriers: safe to leave
  SplitUnit U = split[e];
  const Item it = items[U.first];
  const int n_b = U.n_parts - 1;
  uint32_t bad = 0;
#pragma unroll
  for (int b = 0; b < kMaxSplitParts - 1; ++b) {
    if (b < n_b) {
      const WideBound& B = bounds[U.bnd + b];
      bool diff = false;
#pragma unroll
      for (int v = 0; v < W::V; ++v)
        diff = diff || B.v_end[64 * v + lane] != B.v_start[64 * v + lane];
      if (__ballot(diff) != 0) bad |= 1u << b;
    }
  }
  const int fail = bad ? (int)__builtin_ctz(bad) : -1;
  const int stop = fail < 0 ? n_b : fail;
  int64_t T = bounds[U.bnd].m_end, D = 0;  // part 0 is exact
  for (int b = 0; b < stop; ++b) {
    D = T - bounds[U.bnd + b].m_start;
    if (b + 1 < n_b) T = bounds[U.bnd + b + 1].m_end + D;
  }
  if (fail < 0) {
    if (lane == 0 && metric && it.frame >= 0) metric[it.frame] = last_m[it.slot] + D;
    return;
  }
  if (lane == 0) rep_m0[it.slot] = T;
  __threadfence();
  U.it_begin = units[U.warm + fail + 1].it_begin;
  U.it_end = it.n_stages;
  U.warm = 0;
  U.part = fail + 1;
  const DevCode c = codes[it.code];
  wpk::unit<N, BETA>(c, it, U, 1, bounds, const_cast<int64_t*>(last_m), rep_m0, llr, surv, metric,
                     end_out, item_end, tbl_all[wid], lane);
}

template <int N, int BETA>
static hipError_t wpk_launch(const DevCode* codes, const Item* items, const SplitUnit* units,
                             int n_units, const int8_t* llr, uint64_t* surv, int64_t* metric,
                             int32_t* end_out, int32_t* item_end, WideBound* bounds,
                             int64_t* last_m, const SplitUnit* split, int n_split,
                             int64_t* rep_m0, hipStream_t st) {
  const dim3 block(64 * wpk::kWaves);
  hipLaunchKernelGGL((k_fwd_wpk<N, BETA>), dim3((n_units + wpk::kWaves - 1) / wpk::kWaves), block,
                     0, st, codes, items, units, n_units, bounds, last_m, llr, surv, metric,
                     end_out, item_end);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess || n_split <= 0) return e;
  hipLaunchKernelGGL((k_wpk_check<N, BETA>), dim3((n_split + wpk::kWaves - 1) / wpk::kWaves),
                     block, 0, st, codes, items, split, n_split, units, bounds,
                     (const int64_t*)last_m, rep_m0, llr, surv, metric, end_out, item_end);
  return hipGetLastError();
}

hipError_t launch_fwd_wpk(int K, int beta, const DevCode* codes, const Item* items,
                          const SplitUnit* units, int n_units, const int8_t* llr, uint64_t* surv,
                          int64_t* metric, int32_t* end_out, int32_t* item_end, WideBound* bounds,
                          int64_t* last_m, const SplitUnit* split, int n_split, int64_t* rep_m0,
                          hipStream_t st) {
#define MV_WPK(N, B)                                                                              \
  return wpk_launch<N, B>(codes, items, units, n_units, llr, surv, metric, end_out, item_end,     \
                          bounds, last_m, split, n_split, rep_m0, st)
  switch (K * 8 + beta) {
    case 8 * 8 + 2: MV_WPK(7, 2);
    case 8 * 8 + 3: MV_WPK(7, 3);
    case 9 * 8 + 2: MV_WPK(8, 2);
    case 9 * 8 + 3: MV_WPK(8, 3);
    default: return hipErrorInvalidValue;
  }
#undef MV_WPK
}

}  // namespace mivit

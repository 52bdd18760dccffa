// Forward procedure for int8 soft values, rate 1/2, K = 5 or 7: two frames
// packed in the 16-bit halves of every register, radix-4 survivors.
//
// Trellis (§VIII-A).  One iteration is two stages: it maps the left state
// i = 4f + y to the right state j = f + 2^(n-2) u (n = K-1) and keeps the
// 2-bit decision y.  It runs here as two radix-2 stages whose decisions
// collect in the metric itself: a stage takes two additions and one packed
// maximum per register for both frames, and only every second stage strips
// the collected decision from the metric's low bits.  (Radix 4 in one step
// takes four additions, three maxima and a strip-and-retag.)
//
// Metrics.  A 16-bit half holds 8 (PM + offset) + 3 + h, h the history of the
// current iteration.  A stage's even candidate adds t = 8 m + g and its odd
// candidate subtracts the same t (by the corollary of §IV the two branches
// into a state have opposite metrics m), g = 1 for the first stage of an
// iteration and 2 for the second.  Equal metrics therefore go to the even
// previous state (R1), histories never decide between unequal ones, and
// after both stages 3 + h = 6 - 2y: bits 1 and 2 hold 3 - y.  Both frames
// share one 32-bit addition: t is the sum of frame A's value and 65536 times
// frame B's, both signed; since every half of the true sum lies in [0, 65535]
// no carry or borrow of one half is lost in the other.
//
// Range control.  The metrics of a frame's states never differ by more than
// W = 256 w, w the largest output weight of n stages leaving a common state
// (two paths into any two states can be continued alike up to n stages ago).
// The best metric never falls.  So if state 0 is brought to C = W + 256 every
// REN stages, every metric stays in [C - W, C + W + 256 REN] in between and
// every candidate at 0 or above, which fits 13 bits for REN = 8 and w <= 11
// (the standard K = 7 code has w = 11; K = 5 has w <= 8), and for REN = 4 and
// any K = 7 code.  (From a known start the other states stand below all that
// n stages can make up, so range control waits until stage 8, when every
// state has been reached; the start itself leaves room for that.)  The subtracted
// amounts are accumulated exactly and added back to the final metric.
//
// Positions.  At time t (stages since the first iteration) state s has the
// rotated index r = rotl_n(s, t mod n), so that stage t pairs the indices
// that differ in bit q = t mod n and the new state keeps its index.  Index r
// sits at position p with p0 = r0 ^ r2, p1 = r1 ^ r2 and the other bits
// unchanged; low LB bits of p name the lane, the others the register.  The
// partners of a stage are then the lanes p ^ 1, p ^ 2, p ^ 7 and p ^ 8: each
// one DPP pattern (quad permutations, half-row mirror, row rotation by 8)
// that the subtraction takes as its operand.  (Without the change of
// variables p ^ 4 would take two.)
//   LB = 4: a pair of frames occupies a row of 16 lanes, four pairs a
//     wavefront; K = 7 has four registers per lane, and the stages on the
//     register bits exchange nothing.  For batches that fill the device.
//   LB = 6 (K = 7): one pair per wavefront.  Bits 4 and 5 are a
//     v_permlane16/32_swap of the candidates every lane forms for its own
//     state's two successors.  A short chain for few frames.
//
// Branch metrics.  Per stage a pair has eight table words: t for the four
// output patterns, and -t (for lanes whose own previous state is the odd
// one).  A lane fills one row per block (16 stages; LB = 6: 48), one block
// ahead; kBufs blocks of tables rotate in LDS, entries are read kAhead stages
// ahead, and soft values are loaded kBufs blocks ahead.  Rows are padded so
// that neither the 16-byte stores nor the lookups conflict on LDS banks.
//
// Odd stage counts: stage 0 is evaluated in closed form (the start metrics
// are all zero, or zero at state 0 only); the traceback emits its bit from
// the state at time 1.
//
// Survivors of a pair: per group of 8 iterations 2^n words, word r holding
// 3 - y of iteration 8G + k, frame h (0 = A, 1 = B) in bits
// 16 (k & 1) + 8 h + 2 (k >> 1) and the bit above.
//
// What bounds it: vector issue; four states per lane take 40 instructions per
// iteration, which is 74% of the issue cycles of the large batch's 200 us (two
// wavefronts share a SIMD, and range control, table rows and the reads of the
// entries leave gaps that two do not fill); one state per lane takes 12, 87%.
// Measured, whole decode, against a kernel that took radix 4 in one step:
// K = 7, 4096 frames of 8192 stages 312 -> 251 us (forward 246 -> 203);
// 32768 x 2048 741 -> 540; 1 x 1024 52 -> 31; 2048 x 4096, one pair per
// wavefront, 129 -> 92; K = 5, 4096 x 8192 182 -> 96, 1 x 1024 54 -> 26.  Three
// or four wavefronts per SIMD for the four-state layout were slower: the split
// runs more warm-up stages than the better filling gives.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "mivit_device.h"

namespace mivit {

namespace pk {

constexpr uint32_t kBoth = 0x10001u;
constexpr uint32_t kStrip = 0xFFF8FFF8u;
constexpr uint32_t kTags = 0x06060606u;
// state 0 after range control (metric units): W + 256 for w = 11 and 12
template <int REN>
constexpr int kC = REN == 8 ? 3072 : 3328;
static_assert(8 * (kC<8> + 11 * 256 + 8 * 256) + 7 < 65536, "16-bit range, w <= 11");
static_assert(8 * (kC<4> + 12 * 256 + 4 * 256) + 7 < 65536, "16-bit range, w = 12");
constexpr int kCKnown = 4616;   // state 0 of a known start: above the others by more than
constexpr int kUnreach = 1540;  // what n stages can make up, and these stay above 0 meanwhile
static_assert(kCKnown - kUnreach > 2 * 6 * 256 && kUnreach >= 6 * 256, "unreachable states");
static_assert(8 * (kCKnown + 8 * 256) + 7 < 65536, "16-bit range from a known start");

typedef unsigned short us2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ uint32_t pk_max(uint32_t a, uint32_t b) {
  return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(us2, a),
                                                                __builtin_bit_cast(us2, b)));
}

__device__ __forceinline__ int parity(uint32_t x) { return __popc(x) & 1; }

// beta = 2 output bits of the branch leaving state i on input u (§II-A).
__device__ __forceinline__ int branch_out2(const DevCode& c, int i, int u) {
  const uint32_t reg = ((uint32_t)u << (c.K - 1)) | (uint32_t)i;
  return parity(c.gen[0] & reg) | (parity(c.gen[1] & reg) << 1);
}

__device__ __forceinline__ int rotl_n(int x, int r, int n) {
  return ((x << r) | (x >> (n - r))) & ((1 << n) - 1);
}
__device__ __forceinline__ int rotr_n(int x, int r, int n) { return rotl_n(x, (n - r) % n, n); }

// position <-> rotated index (its own inverse)
__device__ __forceinline__ int index_of(int p) { return p ^ ((p & 4) ? 3 : 0); }

__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Two int8 soft values of one stage; any alignment.
__device__ __forceinline__ uint32_t load_llr2(const int8_t* p) {
  uint16_t w;
  __builtin_memcpy(&w, p, 2);
  return w;
}

// Whether some n-stage path difference has an output weight above 11 (every
// lane weighs one; n = 6).
__device__ __forceinline__ bool wide_spread(const DevCode& c, int lane) {
  int w = 0;
  uint32_t reg = 0;
#pragma unroll
  for (int t = 0; t < 6; ++t) {
    reg |= (uint32_t)((lane >> t) & 1) << 6;
    w += parity(c.gen[0] & reg) + parity(c.gen[1] & reg);
    reg >>= 1;
  }
  return __builtin_amdgcn_ballot_w64(w > 11) != 0;
}

// Metric of the lane that differs in position by bit q's partner pattern.
template <int Q>
__device__ __forceinline__ uint32_t partner(uint32_t x) {
  constexpr int ctrl = Q == 0 ? 0xB1 : Q == 1 ? 0x4E : Q == 2 ? 0x141 : 0x128;
  return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, ctrl, 0xF, 0xF, true);
}

template <int N, int LB>
struct Fwd {
  static constexpr int NS = 1 << N, R = 1 << (N - LB), PAIRS = 64 >> LB;
  static constexpr int kRows = LB == 6 ? 48 : 16;  // stages per table block (a lane fills one)
  static constexpr int kBufs = LB == 6 ? 2 : 3;
  static constexpr int kTrip = kRows * kBufs;      // whole phase periods
  static constexpr int kRow = PAIRS * 8 + 4;       // words per table row (all pairs, padded)
  static constexpr int kBuf = kRows * kRow;        // words per block of tables
  static constexpr int kAhead = R > 1 ? 4 : 8;       // stages an entry is read ahead
  static constexpr bool kSwap = LB == 6;           // bits 4, 5: permlane swaps
  const uint32_t* tp[N][R];  // table entry (row 0, buffer 0) per phase and register
  const uint32_t* tp1[2];    // kSwap: entry of the candidate for input 1, bits 4 and 5
  uint32_t* trow;            // table words this lane fills (buffer 0)
  uint32_t tag;              // g of this lane's row in both halves
  uint32_t strip, three;     // kStrip and 3 * kBoth, in registers: one v_and_or
  const int8_t* l0;          // soft values of stage 0 of iteration 0, frames A and B
  const int8_t* l1;
  uint32_t wa[kBufs], wb[kBufs];  // soft values of this lane's row, blocks ahead
  uint32_t V[R];
  uint32_t q[kAhead][R];     // entries of the stages ahead
  uint32_t q1[kAhead];
  uint32_t v0[R];            // result of the last even iteration
  uint32_t acc[R];           // decisions of the current group
  uint32_t* sv;              // survivor words of the pair, plus this lane's index
  int row;                   // block stage this lane tabulates
  int last;                  // last stage that can be loaded
  int hold;                  // first stage of the trip that skips its range control at stage 4
  // range control: sums of state 0's halves before each, and how many
  uint32_t off0, off1;       // of the current trips
  int64_t sum0, sum1;        // of those before
};

template <int N, int LB>
__device__ __forceinline__ void load(Fwd<N, LB>& F, int b, int stage) {
  const uint64_t x = 2 * (uint64_t)(uint32_t)min(stage + F.row, F.last);
  F.wa[b] = load_llr2(F.l0 + x);
  F.wb[b] = load_llr2(F.l1 + x);
}

// This lane's table row from its soft values, into buffer `buf`.
template <int N, int LB>
__device__ __forceinline__ void table(Fwd<N, LB>& F, int b, int buf) {
  // values + 128, frame A's in the low and frame B's in the high half; the
  // bias cancels in differences, the sum's is in F.tag
  const uint32_t w = (F.wa[b] | (F.wb[b] << 16)) ^ 0x80808080u;
  const uint32_t u0 = w & 0x00FF00FFu, u1 = __builtin_amdgcn_perm(w, w, 0x0C030C01u);
  const uint32_t sum = u1 + u0, dif = u1 - u0;
  constexpr uint32_t bias = 2048u * kBoth;
  const uint32_t T = F.tag;
  const uint32_t e0 = (sum << 3) + (T - bias), e1 = (dif << 3) + T;
  const uint32_t e3 = 2 * T - e0, e2 = 2 * T - e1;
  uint4* dst = (uint4*)(F.trow + buf * F.kBuf);
  dst[0] = make_uint4(e0, e1, e2, e3);
  dst[1] = make_uint4(0u - e0, 0u - e1, 0u - e2, 0u - e3);
}

// Entries of stage K of a trip (K may run into the next trip).
template <int N, int LB, int K>
__device__ __forceinline__ void fetch(Fwd<N, LB>& F) {
  using W = Fwd<N, LB>;
  constexpr int q = K % N, o = (K / W::kRows % W::kBufs) * W::kBuf + (K % W::kRows) * W::kRow;
#pragma unroll
  for (int r = 0; r < W::R; ++r) F.q[K % W::kAhead][r] = F.tp[q][r][o];
  if constexpr (W::kSwap && q >= 4) F.q1[K % W::kAhead] = F.tp1[q - 4][o];
}

// The first kAhead stages' entries.
template <int N, int LB, int K>
__device__ __forceinline__ void first(Fwd<N, LB>& F) {
  if constexpr (K < Fwd<N, LB>::kAhead) {
    fetch<N, LB, K>(F);
    first<N, LB, K + 1>(F);
  }
}

template <int N, int LB, int K>
__device__ __forceinline__ void stage(Fwd<N, LB>& F) {
  using W = Fwd<N, LB>;
  constexpr int Q = K % N, R = W::R;
  uint32_t t[R];
#pragma unroll
  for (int r = 0; r < R; ++r) t[r] = F.q[K % W::kAhead][r];
  if constexpr (W::kSwap && Q >= 4) {
    const uint32_t c0 = F.V[0] + t[0], c1 = F.V[0] + F.q1[K % W::kAhead];
    fetch<N, LB, K + W::kAhead>(F);
    if constexpr (Q == 4) {
      const auto s = __builtin_amdgcn_permlane16_swap(c0, c1, false, false);
      F.V[0] = pk_max(s[0], s[1]);
    } else {
      const auto s = __builtin_amdgcn_permlane32_swap(c0, c1, false, false);
      F.V[0] = pk_max(s[0], s[1]);
    }
  } else {
    fetch<N, LB, K + W::kAhead>(F);
    uint32_t c[R], e[R];
    if constexpr (Q < LB) {
#pragma unroll
      for (int r = 0; r < R; ++r) {
        c[r] = F.V[r] + t[r];
        e[r] = partner<Q>(F.V[r]) - t[r];
      }
    } else {
      constexpr int rb = 1 << (Q - LB);
#pragma unroll
      for (int r = 0; r < R; ++r) {
        c[r] = F.V[r & ~rb] + t[r];
        e[r] = F.V[r | rb] - t[r];
      }
    }
#pragma unroll
    for (int r = 0; r < R; ++r) F.V[r] = pk_max(c[r], e[r]);
  }
}

// Bring state 0 (position 0: register 0 of the pair's lane 0) to kC<REN>;
// `skip`: leave the metrics as they are, and count a subtraction of 0.
template <int N, int LB, int REN>
__device__ __forceinline__ void renorm(Fwd<N, LB>& F, bool skip) {
  constexpr uint32_t target = (uint32_t)(8 * kC<REN> + 3) * kBoth;
  uint32_t ref;
  if constexpr (LB == 6)
    ref = __builtin_amdgcn_readfirstlane(F.V[0]);
  else
    ref = (uint32_t)__builtin_amdgcn_mov_dpp((int)F.V[0], 0x150, 0xF, 0xF, false);  // row lane 0
  ref = skip ? target : ref;
  const uint32_t d = ref - target;  // dA + 65536 dB, both signed 16-bit
#pragma unroll
  for (int r = 0; r < F.R; ++r) F.V[r] -= d;
  F.off0 += ref & 0xFFFFu;
  F.off1 += ref >> 16;
}

// Iteration K/2 of a trip is complete: strip its decisions from the metrics
// and collect them; STORE: write the group's words after its last iteration.
template <int N, int LB, int REN, bool STORE, int K>
__device__ __forceinline__ void iteration_end(Fwd<N, LB>& F, int t0) {
  constexpr int k = (K / 2) & 7;  // iteration of the group
#pragma unroll
  for (int r = 0; r < F.R; ++r) {
    const uint32_t v = F.V[r];
    F.V[r] = (v & F.strip) | F.three;
    if constexpr (STORE) {
      if constexpr ((k & 1) == 0) {
        F.v0[r] = v;
      } else {
        // bytes 0 and 2 of both results: the tags at bits 1, 2 of each byte
        const uint32_t t = __builtin_amdgcn_perm(v, F.v0[r], 0x06040200u) & kTags;
        if constexpr (k == 1) F.acc[r] = t >> 1;
        if constexpr (k == 3) F.acc[r] |= t << 1;
        if constexpr (k == 5) F.acc[r] |= t << 3;
        if constexpr (k == 7) F.acc[r] |= t << 5;
      }
    }
  }
  if constexpr ((K + 1) % REN == 0) renorm<N, LB, REN>(F, REN == 4 && K == 3 && t0 == F.hold);
  if constexpr (STORE && k == 7) {
    uint32_t* dst = F.sv + (int64_t)((t0 + K) >> 4) * F.NS;
#pragma unroll
    for (int r = 0; r < F.R; ++r) dst[16 * r] = F.acc[r];
  }
}

template <int N, int LB, int REN, bool STORE, int K>
__device__ __forceinline__ void step(Fwd<N, LB>& F, int t0) {
  using W = Fwd<N, LB>;
  if constexpr (K % W::kRows == 0) {
    constexpr int b = (K / W::kRows + 1) % W::kBufs;  // the next block
    table(F, b, b);
    load(F, b, t0 + K + (W::kBufs + 1) * W::kRows);
    wave_sync();
  }
  stage<N, LB, K>(F);
  if constexpr (K & 1) iteration_end<N, LB, REN, STORE, K>(F, t0);
}

template <int N, int LB, int REN, bool STORE, int K>
__device__ __forceinline__ void trip(Fwd<N, LB>& F, int t0) {
  if constexpr (K < Fwd<N, LB>::kTrip) {
    step<N, LB, REN, STORE, K>(F, t0);
    // four states per lane: keep each iteration's reads ahead of their stages
    if constexpr ((K & 1) && N - LB == 2) __builtin_amdgcn_sched_barrier(0);
    trip<N, LB, REN, STORE, K + 1>(F, t0);
  }
}

// The last, partial trip: the stages below n (even) from t0; the words of a
// partial group hold zeros for the iterations it lacks.
template <int N, int LB, int REN, int K>
__device__ __forceinline__ void tail(Fwd<N, LB>& F, int t0, int n) {
  if constexpr (K < Fwd<N, LB>::kTrip - 2) {
    if (K < n) {
      step<N, LB, REN, true, K>(F, t0);
      step<N, LB, REN, true, K + 1>(F, t0);
      constexpr int k = (K / 2) & 7;
      if (K + 2 == n) {
        if constexpr (k != 7) {
          uint32_t* dst = F.sv + (int64_t)((t0 + K) >> 4) * F.NS;
#pragma unroll
          for (int r = 0; r < F.R; ++r) {
            uint32_t w = k == 0 ? 0u : F.acc[r];
            if constexpr ((k & 1) == 0) {
              const uint32_t t = __builtin_amdgcn_perm(F.v0[r], F.v0[r], 0x0C0C0200u) & kTags;
              w |= k == 0 ? t >> 1 : t << (k - 1);
            }
            dst[16 * r] = w;
          }
        }
      } else {
        tail<N, LB, REN, K + 2>(F, t0, n);
      }
    }
  }
}

}  // namespace pk

// One wavefront decodes 64 >> LB pairs of frames of equal length: lane group
// m (2^LB lanes) holds frames 2m (low halves) and 2m+1 (high).  It runs the
// iterations of one unit (whole frames, one part of frames split in time, or
// a repair, kind 1).  Split units that are not last leave their end metrics
// in a boundary record; the last part reports the end state and its own
// metric, which the check completes.
template <int N, int LB, int REN>
__device__ __forceinline__ void fwd_pk_unit(const DevCode& c, const Item* __restrict__ items,
                                            const SplitUnit U, int kind, R4Bound* bounds,
                                            int64_t* last_m, const int64_t* rep_m0,
                                            const int8_t* __restrict__ llr,
                                            uint64_t* __restrict__ surv, int64_t* metric,
                                            int32_t* end_out, int32_t* item_end, uint32_t* tbl,
                                            int lane) {
  using namespace pk;
  using W = Fwd<N, LB>;
  constexpr int NS = W::NS, R = W::R, LANES = 1 << LB;
  const int m = lane >> LB, l = lane & (LANES - 1);
  const bool va = 2 * m < U.count, vb = 2 * m + 1 < U.count;
  // a pair beyond the frame count repeats pair 0 (same inputs, same stores),
  // a missing frame B its frame A
  const int ia = U.first + (va ? 2 * m : 0);
  const int ib = va ? (vb ? ia + 1 : ia) : U.first + (U.count > 1 ? 1 : 0);
  const Item ita = items[ia], itb = items[ib];
  const int S = __builtin_amdgcn_readfirstlane(ita.n_stages);  // equal within the wave
  const int lead = S & 1;
  const int t_b = 2 * U.it_begin, t_e = 2 * U.it_end, t_s = 2 * (U.it_begin - U.warm);
  const bool first_part = kind == 0 && U.part == 0;
  const bool split = U.n_parts > 1;

  W F;
  F.row = LB == 6 ? min(lane, W::kRows - 1) : lane & 15;
  F.last = (S >> 1) * 2 - 1;
  F.hold = kind == 0 ? t_s : -1;
  F.trow = tbl + F.row * W::kRow + m * 8;
  F.tag = (uint32_t)((F.row & 1) ? 2 : 1) * kBoth;
  F.l0 = llr + ita.llr_off + 2 * lead;
  F.l1 = llr + itb.llr_off + 2 * lead;
  F.sv = (uint32_t*)(surv + ita.surv_off) + index_of(l);
  // register copies the compiler does not fold back into two literals
  asm volatile("s_mov_b32 %0, %1" : "=s"(F.strip) : "n"(kStrip));
  asm volatile("v_mov_b32 %0, %1" : "=v"(F.three) : "n"(3 * kBoth));
  F.off0 = F.off1 = 0;
  F.sum0 = F.sum1 = 0;
  {
    const uint32_t* pt = tbl + m * 8;
#pragma unroll
    for (int q = 0; q < N; ++q) {
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const int x = index_of(l) + 16 * r;  // rotated index
        const bool odd = (x >> q) & 1;       // the lane's own previous state is the odd one
        if (W::kSwap && q >= 4) {
          // candidates of the lane's own state for inputs 0 and 1
          const int p0 = branch_out2(c, rotr_n(x, q, N), 0);
          F.tp[q][r] = pt + (odd ? 4 + (3 ^ p0) : p0);
          F.tp1[q - 4] = pt + (odd ? 4 + p0 : 3 ^ p0);
        } else {
          const int j = rotr_n(x, (q + 1) % N, N);
          const int pe = branch_out2(c, (j << 1) & (NS - 1), j >> (N - 1));
          F.tp[q][r] = pt + (q < LB && odd ? 4 + pe : pe);
        }
      }
    }
  }

  // metrics entering iteration t_s / 2: at a multiple of the trip, so the
  // rotated index is the state
  int c_init = kC<REN>;
  if (first_part) {
    const Item* its[2] = {&ita, &itb};
    if (ita.start_known || itb.start_known) c_init = kCKnown;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int j = index_of(l) + 16 * r;
      uint32_t v[2];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const bool known = its[h]->start_known != 0;
        int pm = 0;
        bool reach = !known || j == 0;
        if (lead) {
          const int8_t* p = llr + its[h]->llr_off;
          const int i0 = (j << 1) & (NS - 1);
          const int w = branch_out2(c, i0, j >> (N - 1));
          const int bm = ((w & 1) ? -(int)p[0] : (int)p[0]) + ((w & 2) ? -(int)p[1] : (int)p[1]);
          reach = !known || i0 == 0;
          pm = known ? bm : (bm < 0 ? -bm : bm);  // unknown start: max(bm, -bm)
        }
        v[h] = 8u * (uint32_t)(reach ? c_init + pm : kUnreach) + 3u;
      }
      F.V[r] = v[0] | (v[1] << 16);
    }
  } else if (kind == 0) {
#pragma unroll
    for (int r = 0; r < R; ++r) F.V[r] = (uint32_t)(8 * kC<REN> + 3) * kBoth;  // unknown start
  } else {
    const R4Bound& B = bounds[U.bnd + U.part - 1];
#pragma unroll
    for (int r = 0; r < R; ++r) F.V[r] = B.v_end[64 * r + lane];  // repair
  }
  // subtracted up to stage t, in metric units, per half
  auto taken = [&](int h, int t) -> int64_t {
    const int64_t n = (t - t_s) / REN;
    return ((h ? F.sum1 + F.off1 : F.sum0 + F.off0) - n * (8 * kC<REN> + 3)) / 8;
  };
  // metric of state 0 from this unit's origin where range control has just run
  auto m0 = [&](int h, int t) -> int64_t { return kC<REN> - c_init + taken(h, t); };
  if (t_e > t_s) {
#pragma unroll
    for (int b = 0; b < W::kBufs; ++b) load(F, b, t_s + W::kRows * b);
    table(F, 0, 0);
    load(F, 0, t_s + W::kBufs * W::kRows);
    wave_sync();
    first<N, LB, 0>(F);
    auto flush = [&]() {
      F.sum0 += F.off0;
      F.sum1 += F.off1;
      F.off0 = F.off1 = 0;
    };
    // (only where wavefronts share SIMDs)
    const int slot = gridDim.x > kComputeUnits ? wave_slot() : -1;
    int t0 = t_s;
    for (; t0 < t_b; t0 += W::kTrip) trip<N, LB, REN, false, 0>(F, t0);  // warm-up: no stores
    if (kind == 0 && U.part > 0) {
      R4Bound& B = bounds[U.bnd + U.part - 1];
#pragma unroll
      for (int r = 0; r < R; ++r) B.v_start[64 * r + lane] = F.V[r];
      if (l == 0) {
        B.m_start[2 * m] = m0(0, t_b);
        B.m_start[2 * m + 1] = m0(1, t_b);
      }
    }
    for (; t0 + W::kTrip <= t_e; t0 += W::kTrip) {
      if (slot >= 0) fair_share(slot, (t0 - t_s) / W::kTrip);
      trip<N, LB, REN, true, 0>(F, t0);
      flush();
    }
    if (t0 < t_e) tail<N, LB, REN, 0>(F, t0, t_e - t0);
  }
  if (kind == 0 && split && U.part < U.n_parts - 1) {
    R4Bound& B = bounds[U.bnd + U.part];
#pragma unroll
    for (int r = 0; r < R; ++r) B.v_end[64 * r + lane] = F.V[r];
    if (l == 0) {
      B.m_end[2 * m] = m0(0, t_e);
      B.m_end[2 * m + 1] = m0(1, t_e);
    }
    return;
  }

  // final metrics: index r holds state rotr(r, t_e mod n)
  const int rot = t_e % N;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const Item& it = h ? itb : ita;
    const bool valid = h ? vb : va;
    uint32_t val[R];
    uint32_t key = 0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      val[r] = (F.V[r] >> (16 * h)) & 0xFFFFu;
      const int s = rotr_n(index_of(l) + 16 * r, rot, N);
      const uint32_t k = (val[r] << 8) | (uint32_t)(255 - s);
      key = k > key ? k : key;
    }
#pragma unroll
    for (int o = 1; o < LANES; o <<= 1) {
      const uint32_t other = (uint32_t)__shfl_xor((int)key, o);
      key = other > key ? other : key;
    }
    const bool fixed = it.end_state >= 0;
    const int js = fixed ? it.end_state : 255 - (int)(key & 255);
    const int x = rotl_n(js & (NS - 1), rot, N);
    uint32_t vfix = 0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int src = LANES * m + index_of(R > 1 ? x & 15 : x);
      const uint32_t y = (uint32_t)__shfl((int)val[r], src);
      vfix = (R == 1 || (x >> 4) == r) ? y : vfix;
    }
    const uint32_t vbest = fixed ? vfix : key >> 8;
    if (l == 0 && valid) {
      item_end[it.slot] = js;
      const int64_t local = (int64_t)(vbest >> 3) - c_init + taken(h, t_e);
      if (kind == 0 && split) {
        last_m[it.slot] = local;  // completed by the check
        if (it.frame >= 0 && end_out) end_out[it.frame] = js;
      } else if (it.frame >= 0) {
        if (end_out) end_out[it.frame] = js;
        if (metric) metric[it.frame] = local + (kind == 1 ? rep_m0[it.slot] : 0);
      }
    }
  }
}

template <int N, int LB>
__device__ __forceinline__ void fwd_pk_wave(const DevCode* __restrict__ codes,
                                            const Item* __restrict__ items, const SplitUnit U,
                                            int kind, R4Bound* bounds, int64_t* last_m,
                                            const int64_t* rep_m0,
                                            const int8_t* __restrict__ llr,
                                            uint64_t* __restrict__ surv, int64_t* metric,
                                            int32_t* end_out, int32_t* item_end, uint32_t* tbl,
                                            int lane) {
  // one code per part
  const DevCode c = codes[__builtin_amdgcn_readfirstlane(items[U.first].code)];
  if (N == 6 && pk::wide_spread(c, lane))
    fwd_pk_unit<N, LB, 4>(c, items, U, kind, bounds, last_m, rep_m0, llr, surv, metric, end_out,
                          item_end, tbl, lane);
  else
    fwd_pk_unit<N, LB, 8>(c, items, U, kind, bounds, last_m, rep_m0, llr, surv, metric, end_out,
                          item_end, tbl, lane);
}

constexpr int kPkWaves = 4;  // wavefronts per workgroup, one per SIMD (they share nothing)
// Table buffers reserved per wavefront.  A pair per wavefront uses two; the room of
// the third keeps its workgroups from crowding out those of other codes in a
// mixed batch (10000 frames of K = 5, 7, 9: 609 us, 624 without it), and alone
// it makes no difference.
constexpr int kTblBufs = 3;

// One wavefront per unit, or (counter != nullptr) a persistent grid whose
// wavefronts take units in table order from a device counter that starts at
// zero, until the table is exhausted.
template <int N, int LB>
__global__ __launch_bounds__(64 * kPkWaves, N - LB == 2 ? 2 : 4) void k_fwd_pk(
    const DevCode* __restrict__ codes, const Item* __restrict__ items,
    const SplitUnit* __restrict__ units, int n_units, R4Bound* bounds, int64_t* last_m,
    const int8_t* __restrict__ llr, uint64_t* __restrict__ surv, int64_t* metric,
    int32_t* end_out, int32_t* item_end, int32_t* counter) {
  __shared__ __align__(16) uint32_t tbl_all[kPkWaves][kTblBufs * pk::Fwd<N, LB>::kBuf];
  const int wid = threadIdx.x >> 6;
  const int lane = threadIdx.x & 63;
  int u = __builtin_amdgcn_readfirstlane(blockIdx.x * kPkWaves + wid);
  for (;;) {
    if (counter) {
      int w = 0;
      if (lane == 0) w = atomicAdd(counter, 1);
      u = __builtin_amdgcn_readfirstlane(w);
    }
    if (u >= n_units) return;  // no workgroup barriers: safe to leave
    fwd_pk_wave<N, LB>(codes, items, units[u], 0, bounds, last_m, nullptr, llr, surv, metric,
                       end_out, item_end, tbl_all[wid], lane);
    if (!counter) return;
  }
}

// The check after a split forward pass, one wavefront per split entry (its
// part-0 unit): boundary k is exact when part k's metrics at its end equal
// part k+1's after its warm-up at every position (both are range-controlled
// to state 0 there, so equal words mean metric vectors that differ by a
// constant).  Every boundary of the entry is loaded at once.  Lane k
// follows frame k of the entry: T = the true metric of state 0 at the first
// inexact boundary, D = the constant the last part's metrics lack when all
// are exact.
struct EntryCheck {
  int fail;  // first inexact boundary, or -1
  int64_t T, D;
};

template <int NV>
__device__ __forceinline__ EntryCheck check_entry(const SplitUnit& U,
                                                  const R4Bound* __restrict__ bounds, int lane) {
  const int n_b = U.n_parts - 1;
  const int k = lane < U.count ? lane : 0;
  uint32_t bad = 0;
#pragma unroll
  for (int b = 0; b < kMaxSplitParts - 1; ++b) {
    if (b < n_b) {
      const R4Bound& B = bounds[U.bnd + b];
      bool diff = false;
#pragma unroll
      for (int x = 0; x < NV / 64; ++x) diff = diff || B.v_end[64 * x + lane] != B.v_start[64 * x + lane];
      if (__ballot(diff) != 0) bad |= 1u << b;
    }
  }
  EntryCheck r;
  r.fail = bad ? (int)__builtin_ctz(bad) : -1;
  const int last = r.fail < 0 ? n_b : r.fail;
  int64_t T = bounds[U.bnd].m_end[k], D = 0;  // part 0 is exact
  for (int b = 0; b < last; ++b) {
    D = T - bounds[U.bnd + b].m_start[k];
    if (b + 1 < n_b) T = bounds[U.bnd + b + 1].m_end[k] + D;
  }
  r.T = T;
  r.D = D;
  return r;
}

// The repair unit of an entry whose boundary `fail` is inexact: the frames
// from that boundary to their end, from the metrics part `fail` left there.
__device__ __forceinline__ SplitUnit repair_unit(const SplitUnit& U, const SplitUnit* units,
                                                 int fail, int n_stages) {
  SplitUnit R = U;
  R.it_begin = units[U.warm + fail + 1].it_begin;
  R.it_end = n_stages >> 1;
  R.warm = 0;
  R.part = fail + 1;
  return R;
}

// Check of the split entries; an entry with an inexact boundary is repaired
// by the same wavefront, right here.
template <int N, int LB>
__global__ __launch_bounds__(64 * kPkWaves, N - LB == 2 ? 2 : 4) void k_pk_check(
    const DevCode* __restrict__ codes, const Item* __restrict__ items,
    const SplitUnit* __restrict__ split, int n_split, const SplitUnit* __restrict__ units,
    R4Bound* bounds, const int64_t* __restrict__ last_m, int64_t* rep_m0,
    const int8_t* __restrict__ llr, uint64_t* __restrict__ surv, int64_t* metric,
    int32_t* end_out, int32_t* item_end) {
  __shared__ __align__(16) uint32_t tbl_all[kPkWaves][kTblBufs * pk::Fwd<N, LB>::kBuf];
  const int wid = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int e = __builtin_amdgcn_readfirstlane(blockIdx.x * kPkWaves + wid);
  if (e >= n_split) return;  // no workgroup barriers: safe to leave
  const SplitUnit U = split[e];
  const EntryCheck c = check_entry<64 * pk::Fwd<N, LB>::R>(U, bounds, lane);
  const bool mine = lane < U.count;
  const Item it = items[U.first + (mine ? lane : 0)];
  if (c.fail < 0) {
    if (mine && metric && it.frame >= 0) metric[it.frame] = last_m[it.slot] + c.D;
    return;
  }
  if (mine) rep_m0[it.slot] = c.T;
  __threadfence();
  fwd_pk_wave<N, LB>(codes, items, repair_unit(U, units, c.fail, items[U.first].n_stages), 1,
                     bounds, const_cast<int64_t*>(last_m), rep_m0, llr, surv, metric, end_out,
                     item_end, tbl_all[wid], lane);
}

// Forward pass of a part; split entries are then checked (and repaired in
// place) by one more launch.
template <int N, int LB>
hipError_t pk_launch(const DevCode* codes, const Item* items, const SplitUnit* units, int n_units,
                     const int8_t* llr, uint64_t* surv, int64_t* metric, int32_t* end_out,
                     int32_t* item_end, int32_t* counter, int grid_limit, R4Bound* bounds,
                     int64_t* last_m, const SplitUnit* split, int n_split, int64_t* rep_m0,
                     hipStream_t st) {
  if (n_units <= 0) return hipSuccess;
  const int threads = 64 * kPkWaves;
  int nb = (n_units + kPkWaves - 1) / kPkWaves;
  if (counter) {
    const int lim = grid_limit > 0 ? grid_limit : resident_workgroups(k_fwd_pk<N, LB>, threads);
    if (lim > 0 && nb > lim) nb = lim;
  }
  hipLaunchKernelGGL((k_fwd_pk<N, LB>), dim3(nb), dim3(threads), 0, st, codes, items, units,
                     n_units, bounds, last_m, llr, surv, metric, end_out, item_end, counter);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || n_split <= 0) return e;
  const int ns = (n_split + kPkWaves - 1) / kPkWaves;
  hipLaunchKernelGGL((k_pk_check<N, LB>), dim3(ns), dim3(threads), 0, st, codes, items, split,
                     n_split, units, bounds, (const int64_t*)last_m, rep_m0, llr, surv, metric,
                     end_out, item_end);
  return hipGetLastError();
}

// One state per lane: K = 7 (one pair of frames per wavefront) or K = 5
// (four).
hipError_t launch_fwd_r4p(int K, const DevCode* codes, const Item* items, const SplitUnit* units,
                          int n_units, const int8_t* llr, uint64_t* surv, int64_t* metric,
                          int32_t* end_out, int32_t* item_end, int32_t* counter, int grid_limit,
                          R4Bound* bounds, int64_t* last_m, const SplitUnit* split, int n_split,
                          int64_t* rep_m0, hipStream_t st) {
  if (K != 5 && K != 7) return hipErrorInvalidValue;
  return K == 7 ? pk_launch<6, 6>(codes, items, units, n_units, llr, surv, metric, end_out,
                                  item_end, counter, grid_limit, bounds, last_m, split, n_split,
                                  rep_m0, st)
                : pk_launch<4, 4>(codes, items, units, n_units, llr, surv, metric, end_out,
                                  item_end, counter, grid_limit, bounds, last_m, split, n_split,
                                  rep_m0, st);
}

// Four states per lane: K = 7, four pairs per wavefront.
hipError_t launch_fwd_r4q(const DevCode* codes, const Item* items, const SplitUnit* units,
                          int n_units, const int8_t* llr, uint64_t* surv, int64_t* metric,
                          int32_t* end_out, int32_t* item_end, int32_t* counter, int grid_limit,
                          R4Bound* bounds, int64_t* last_m, const SplitUnit* split, int n_split,
                          int64_t* rep_m0, hipStream_t st) {
  return pk_launch<6, 4>(codes, items, units, n_units, llr, surv, metric, end_out, item_end,
                         counter, grid_limit, bounds, last_m, split, n_split, rep_m0, st);
}

}  // namespace mivit

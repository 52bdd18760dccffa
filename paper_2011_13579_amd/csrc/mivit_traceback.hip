// Parallel traceback (Algorithm 2): frames are cut into segments, one lane
// each, traced at the same time and checked against each other.
//
// The lane whose chase reaches the item's last stage starts from the true
// final state and is exact.  Every other lane starts some stages above its
// segment from a guessed state; survivor paths merge quickly going backwards,
// so it usually meets the true path before reaching its segment.  Exactness
// does not rest on that: lane g records the state y_g it passes at its
// segment's upper boundary and its final state x_g at the lower boundary.
// When y_g equals x_{g+1} of the lane above (itself exact), lane g followed
// the true path through its whole segment.  A ballot finds the lanes where
// this fails; they trace again from x_{g+1} and the check repeats until every
// boundary agrees.
//
// Survivor words are staged through LDS (global_load_lds, no register
// staging), double buffered: the lanes advance in lockstep rounds, the next
// round's words streaming in while the current round is chased.
//
// k_tb_rot reads the survivors of the rotating and packed kernels (every
// default), k_tb_seg those of the generic kernels.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "mivit_device.h"

namespace mivit {

// survivor layouts
enum : int {
  kLayoutNatR2 = 0,  // per stage, ceil(NS/64) uint64 words, bit j = decision of state j
  kLayoutNatR4 = 1,  // same words; stage pairs (t, t+1) from 0 hold bits 0 and 1 of y
  kLayoutNatR8 = 5,  // same words; stage triples (t, t+1, t+2) from 0 hold bits 0..2 of y,
                     // the S mod 3 last stages radix-2 decisions
};

template <int LAYOUT>
struct TbGeom {
  int K, KM1, NS, W;  // W: uint64 words per stage (natural layouts)
  int SB;             // stages per block
  int WB;             // uint32 words per block
  __device__ TbGeom(int K_) : K(K_), KM1(K_ - 1), NS(1 << (K_ - 1)) {
    W = words_per_stage(K_);
    if (LAYOUT == kLayoutNatR8) {
      SB = (32 / W) / 3 * 3;  // whole triples per block: 30, 15 or 6 stages
      WB = SB * 2 * W;
    } else {
      SB = 32 / W;
      WB = 64;
    }
  }
};

typedef __attribute__((address_space(3))) void* lds_ptr_t;

// Stream this lane's 64-word block starting at src into LDS buffer buf_k
// (for the lanes currently active): word w of lane l sits at ((w/4)*64 + l)*4
// + w%4, the layout one 16-byte global_load_lds per lane and chunk produces.  Always 64 words: a block of fewer words
// is followed by more survivor words or by the allocation's padding.
__device__ __forceinline__ void fetch_block(const uint32_t* src, uint32_t* buf_k) {
#pragma unroll
  for (int c = 0; c < 16; ++c)
    __builtin_amdgcn_global_load_lds((const void*)(src + 4 * c), (lds_ptr_t)(buf_k + c * 256),
                                     16, 0, 0);
}

__device__ __forceinline__ uint32_t word_at(const uint32_t* buf_k, int w, int lane) {
  return buf_k[((w >> 2) * 64 + lane) * 4 + (w & 3)];
}

// Per-lane chase state.  Times are stage boundaries: time t is the state
// entering stage t.  In the natural radix-4 layout the decisions of a stage
// pair (2k, 2k+1) only name the state two stages back, so states are known
// (and compared between segments) at pair-aligned times: even times and S.
// In the radix-8 layout they are the multiples of 3 and the times of the
// radix-2 stages at the end.
struct Chase {
  int top, a, b;  // from time top down to time a; bits of [a, b) are emitted
  int j;          // current state
  int xa, yb;     // pair-aligned times at or above a and b
  int x, y;       // states at times xa and yb
};

// All lanes with go set chase their range; the others idle.  Returns with
// c.j = state where the chase ended, c.x and c.y set.
template <int LAYOUT>
__device__ __forceinline__ void chase_all(const TbGeom<LAYOUT>& g, const uint32_t* __restrict__ sv,
                                          uint32_t* lds, Chase& c, bool go, int ob, int S,
                                          uint32_t* bits, int64_t bit_off) {
  const int lane = threadIdx.x;
  const int SB = g.SB, WB = g.WB;
  GroupEmitter em;
  if (go && c.top == c.yb) c.y = c.j;
  if (go && c.top == c.xa) c.x = c.j;
  const int B0 = go ? (c.top - 1) / SB : 0;
  const int nb = go ? B0 - c.a / SB + 1 : 0;
  int t = c.top - 1;  // next stage to step over
  if (nb > 0) fetch_block(sv + (int64_t)B0 * WB, lds);
  for (int r = 0;; ++r) {
    if (__ballot(r < nb) == 0) break;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    uint32_t* cur = lds + (r & 1) * 4096;
    uint32_t* nxt = lds + ((r + 1) & 1) * 4096;
    if (r + 1 < nb) fetch_block(sv + (int64_t)(B0 - r - 1) * WB, nxt);
    if (r < nb) {
      const int B = B0 - r;
      const int t0 = B * SB;  // first stage of the block: t - t0 = t mod SB
      int j = c.j;
      if (LAYOUT == kLayoutNatR4) {
        if ((S & 1) && t == S - 1 && t >= t0) {
          // odd stage count: the last stage was a radix-2 stage
          const int w = (t - t0) * 2 * g.W + (j >> 5);
          const int d = (word_at(cur, w, lane) >> (j & 31)) & 1;
          if (t >= c.a && t < c.b) em.put(t - ob, (uint32_t)(j >> (g.KM1 - 1)), bits, bit_off);
          j = ((j << 1) | d) & (g.NS - 1);
          if (t == c.yb) c.y = j;
          if (t == c.xa) c.x = j;
          --t;
        }
        // pairs (t-1, t), t odd; pairs never straddle a block
        for (; t > t0 && t >= c.a; t -= 2) {
          const int w0 = (t - 1 - t0) * 2 * g.W + (j >> 5);
          const int w1 = (t - t0) * 2 * g.W + (j >> 5);
          const int yy = ((word_at(cur, w0, lane) >> (j & 31)) & 1) |
                         (((word_at(cur, w1, lane) >> (j & 31)) & 1) << 1);
          if (t < c.b) em.put(t - ob, (uint32_t)(j >> (g.KM1 - 1)), bits, bit_off);
          if (t - 1 >= c.a && t - 1 < c.b)
            em.put(t - 1 - ob, (uint32_t)((j >> (g.KM1 - 2)) & 1), bits, bit_off);
          j = 4 * (j & ((g.NS >> 2) - 1)) + yy;
          if (t - 1 == c.yb) c.y = j;
          if (t - 1 == c.xa) c.x = j;
        }
      } else if (LAYOUT == kLayoutNatR8) {
        // the S mod 3 last stages were radix-2 stages
        for (; t >= S - S % 3 && t >= t0 && t >= c.a; --t) {
          const int w = (t - t0) * 2 * g.W + (j >> 5);
          const int d = (word_at(cur, w, lane) >> (j & 31)) & 1;
          if (t < c.b) em.put(t - ob, (uint32_t)(j >> (g.KM1 - 1)), bits, bit_off);
          j = ((j << 1) | d) & (g.NS - 1);
          if (t == c.yb) c.y = j;
          if (t == c.xa) c.x = j;
        }
        // triples (t-2, t-1, t), t = 2 mod 3; triples never straddle a block
        for (; t >= t0 + 2 && t >= c.a; t -= 3) {
          const int sh = j & 31;
          const int w2 = (t - t0) * 2 * g.W + (j >> 5);
          const int w1 = w2 - 2 * g.W, w0 = w1 - 2 * g.W;
          const int yy = ((word_at(cur, w0, lane) >> sh) & 1) |
                         (((word_at(cur, w1, lane) >> sh) & 1) << 1) |
                         (((word_at(cur, w2, lane) >> sh) & 1) << 2);
          if (t < c.b) em.put(t - ob, (uint32_t)(j >> (g.KM1 - 1)), bits, bit_off);
          if (t - 1 >= c.a && t - 1 < c.b)
            em.put(t - 1 - ob, (uint32_t)((j >> (g.KM1 - 2)) & 1), bits, bit_off);
          if (t - 2 >= c.a && t - 2 < c.b)
            em.put(t - 2 - ob, (uint32_t)((j >> (g.KM1 - 3)) & 1), bits, bit_off);
          j = 8 * (j & ((g.NS >> 3) - 1)) + yy;
          if (t - 2 == c.yb) c.y = j;
          if (t - 2 == c.xa) c.x = j;
        }
      } else {
        const int lo = max(c.a, t0);
        for (; t >= lo; --t) {
          const int w = (t - t0) * 2 * g.W + (j >> 5);
          const int d = (word_at(cur, w, lane) >> (j & 31)) & 1;
          if (t < c.b) em.put(t - ob, (uint32_t)(j >> (g.KM1 - 1)), bits, bit_off);
          j = ((j << 1) | d) & (g.NS - 1);
          if (t == c.yb) c.y = j;
          if (t == c.xa) c.x = j;
        }
      }
      c.j = j;
    }
  }
  em.flush(bits);
}

template <int LAYOUT>
__global__ __launch_bounds__(64) void k_tb_seg(const DevCode* __restrict__ codes,
                                               const Item* __restrict__ items,
                                               const uint64_t* __restrict__ surv,
                                               const int32_t* __restrict__ item_end,
                                               uint32_t* __restrict__ bits, int warm) {
  __shared__ uint32_t lds[2 * 4096];
  const Item it = items[blockIdx.x];
  if (it.n_out <= 0) return;
  const DevCode code = codes[it.code];
  const TbGeom<LAYOUT> g(code.K);
  const int lane = threadIdx.x;
  const uint32_t* sv = (const uint32_t*)(surv + it.surv_off);
  const int S = it.n_stages, ob = it.out_begin, n = it.n_out;
  // the next time at or above t where states are known (every time for
  // radix 2; even times and S for radix 4; multiples of 3 and the times from
  // S - S mod 3 on for radix 8)
  auto align = [&](int t) {
    if (LAYOUT == kLayoutNatR4) return ((t & 1) && t < S) ? t + 1 : t;
    if (LAYOUT == kLayoutNatR8) return (t % 3 && t < S - S % 3) ? t + 3 - t % 3 : t;
    return t;
  };
  // segment geometry: G segments of L stages, L a multiple of 32
  int G = min(64, (n + 31) / 32);
  const int L = (((n + G - 1) / G) + 31) & ~31;
  G = (n + L - 1) / L;
  const bool active = lane < G;
  Chase c;
  c.a = ob + lane * L;
  c.b = min(ob + (lane + 1) * L, ob + n);
  c.xa = align(c.a);
  c.yb = align(c.b);
  c.top = active ? ((lane == G - 1) ? S : min(S, align(c.b + warm))) : c.a;
  const bool exact = active && c.top == S;
  c.j = exact ? item_end[it.slot] : 0;
  c.x = c.y = -1;
  chase_all<LAYOUT>(g, sv, lds, c, active && c.top > c.a, ob, S, bits, it.bit_off);
  // repair rounds: lane g is right when its state at yb equals lane g+1's
  // state at its xa (the same time)
  for (int round = 0; round <= G; ++round) {
    const int x_up = __shfl_down(c.x, 1) & (g.NS - 1);
    const bool bad = active && !exact && lane < G - 1 && c.y != x_up;
    if (__ballot(bad) == 0) break;
    // lanes that agree with their neighbour stay idle this round
    Chase r = c;
    r.top = c.yb;
    r.j = x_up;
    chase_all<LAYOUT>(g, sv, lds, r, bad, ob, S, bits, it.bit_off);
    if (bad) {
      c.j = r.j;
      c.x = r.x;
      c.y = x_up;
    }
  }
}

hipError_t launch_tb_seg(int layout, const DevCode* codes, const Item* items, int n_items,
                         const uint64_t* surv, const int32_t* item_end, uint32_t* bits,
                         int warm, hipStream_t st) {
  if (n_items <= 0) return hipSuccess;
  dim3 grid(n_items), block(64);
  switch (layout) {
    case kLayoutNatR2:
      hipLaunchKernelGGL(k_tb_seg<kLayoutNatR2>, grid, block, 0, st, codes, items, surv,
                         item_end, bits, warm);
      break;
    case kLayoutNatR4:
      hipLaunchKernelGGL(k_tb_seg<kLayoutNatR4>, grid, block, 0, st, codes, items, surv,
                         item_end, bits, warm);
      break;
    case kLayoutNatR8:
      hipLaunchKernelGGL(k_tb_seg<kLayoutNatR8>, grid, block, 0, st, codes, items, surv,
                         item_end, bits, warm);
      break;
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Traceback of the rotating layouts.
//
// In all of them the state s at time t sits at position rotl_n(s, t mod n),
// n = K-1, and a step down over a stage replaces position bit t mod n by the
// stage's decision (packed radix 4: two stages replace a 2-bit digit).  The
// message bit of stage t is bit t mod n of the position at time t + 1, which
// is the decision that was put there n stages above, at stage t + n.  So a
// lane collects the raw decisions D of 32 stages in a word, and the message
// bits are those words shifted by n: E_b = (D_{b+1} : D_b) >> n.
//
// What bounds it.  A step is a chain: LDS read, bit extract, one bit-select
// that forms the next LDS address.  The position is therefore held as that
// address (the lane's slot and the buffer included), with the address bit of
// every phase in a register; 32 stages are straight-line code with constant
// bit numbers, 3 VALU instructions and one LDS read per stage (two stages for
// packed radix 4) against about 35 VALU instructions and several branches
// when bits were emitted one by one.  Bandwidth is the other bound: every
// lane streams its warm-up as well as its segment, so a batch with enough
// frames is cut into few, long segments (tb_shape).
//
// kWords: rotating radix 2 (K <= 7), per 32 stages 2^n words, word p the
//   decisions at position p, stage t at bit 31 - (t mod 32).
// kBytes: K = 8, 9, per 8 stages 2^n bytes, stage 8g + i at bit 7 - i.
// kDigits: packed K = 8, 9, per 8 stages 2^n bytes, position p at byte
//   (p mod 64) 2^(n-6) + (p >> 6), the radix-4 digit of iteration i in bits
//   6 - 2i and up.
// kPairs: packed radix 4, per frame pair and 8 iterations 2^n words:
//   iteration k of the group, frame h in byte 2 (k & 1) + h, bits
//   2 (k >> 1) and up, holding 3 - digit.  Lanes l and l + 32 trace the two
//   frames of a pair and share its staged words.
// ---------------------------------------------------------------------------
namespace tb {

constexpr int kPairs = kTbPairs, kWords = kTbWords, kBytes = kTbBytes, kDigits = kTbDigits;

template <int KIND, int N>
struct Geo {
  static constexpr int NS = 1 << N;
  // stages per round (one staged buffer) and rounds per 32-stage block
  static constexpr int RS = KIND == kWords ? 32 : KIND >= kBytes ? 2048 / NS : (N == 6 ? 16 : 32);
  static constexpr int RPB = 32 / RS;
  static constexpr int WPR = KIND == kWords ? NS : KIND >= kBytes ? 64 : (N == 6 ? 64 : 32);
  static constexpr int SLOTS = KIND == kPairs ? 32 : 64;  // staged blocks per buffer
  static constexpr int BUF = WPR * 4 * SLOTS;             // bytes per buffer
  static constexpr int CH = WPR / 4 * SLOTS / 64;         // 16-byte loads per lane and round
  static constexpr int STEP = KIND == kPairs || KIND == kDigits ? 2 : 1;  // stages per step
  static constexpr int NP = N % STEP ? N : N / STEP;                      // phases
  static constexpr int NR = N - 6;  // kDigits: position bits below the lane's
  // address offset of position p, and where position bit q sits in it
  __device__ static int off(int p) {
    if (KIND == kWords) return ((p & 3) << 2) | ((p >> 2) << 10);
    if (KIND == kBytes) return (p & 15) | ((p >> 4) << 10);
    if (KIND == kDigits) {
      const int b = ((p & 63) << NR) | (p >> 6);
      return (b & 15) | ((b >> 4) << 10);
    }
    return ((p & 3) << 2) | (((p >> 2) & 1) << 9) | ((p >> 3) << 10);
  }
  __device__ static int pos(int a) {
    if (KIND == kWords) return ((a >> 2) & 3) | (((a >> 10) << 2) & (NS - 1));
    if (KIND == kBytes) return (a & 15) | (((a >> 10) << 4) & (NS - 1));
    if (KIND == kDigits) {
      const int b = (a & 15) | (((a >> 10) << 4) & (NS - 1));
      return (b >> NR) | ((b & ((1 << NR) - 1)) << 6);
    }
    return ((a >> 2) & 3) | (((a >> 9) << 2) & (NS - 1));
  }
  __device__ static int bit(int q) {
    if (KIND == kWords) return q < 2 ? q + 2 : q + 8;
    if (KIND == kBytes) return q < 4 ? q : q + 6;
    if (KIND == kDigits) {
      const int b = q < 6 ? q + NR : q - 6;
      return b < 4 ? b : b + 6;
    }
    return q < 2 ? q + 2 : q + 7;
  }
};

__device__ __forceinline__ int rotl_n(int x, int r, int n) {
  return ((x << r) | (x >> (n - r))) & ((1 << n) - 1);
}

// Output words of one lane, from the highest down, held until the aligned
// group of four they belong to is complete (or the chase ends) and stored
// together: 16-byte pieces instead of partial-line writes spread over the
// chase.
struct WordGroup {
  uint32_t q[4] = {0, 0, 0, 0};
  uint32_t valid = 0;
  uint32_t* base = nullptr;
  __device__ __forceinline__ void flush() {
    if (valid == 15u && ((uintptr_t)base & 15) == 0) {
      *(uint4*)base = make_uint4(q[0], q[1], q[2], q[3]);
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if ((valid >> i) & 1u) base[i] = q[i];
    }
    valid = 0;
  }
  __device__ __forceinline__ void put(uint32_t* out, int k, uint32_t w) {
    base = out + (k & ~3);
#pragma unroll
    for (int i = 0; i < 4; ++i) q[i] = (k & 3) == i ? w : q[i];
    valid |= 1u << (k & 3);
    if ((k & 3) == 0) flush();
  }
};

// Position-address of the predecessor, and the step's decision, for one step
// at stage index i (static) of the block; m, sh: mask and shift of the phase
// (kDigits: the masks of the digit's two bits).
template <int KIND, int N, int I>
__device__ __forceinline__ void step(const char* lds, uint32_t& A, uint32_t m, uint32_t sh,
                                     uint32_t& D) {
  if constexpr (KIND == kWords) {
    const uint32_t w = *(const uint32_t*)(lds + A);
    const uint32_t d = (uint32_t)((int32_t)(w << I) >> 31);  // 0 or ~0
    A = (A & ~m) | (d & m);
    D = (D << 1) + d;  // minus the decisions
  } else if constexpr (KIND == kBytes) {
    constexpr int R = I % Geo<KIND, N>::RS;
    const uint32_t w = *(const uint8_t*)(lds + A + (R >> 3) * Geo<KIND, N>::NS * 64);
    const uint32_t d = (uint32_t)((int32_t)(w << (24 + (R & 7))) >> 31);
    A = (A & ~m) | (d & m);
    D = (D << 1) + d;
  } else if constexpr (KIND == kDigits) {
    // I: iteration of the round; byte I >> 2 of the position
    constexpr int b = 6 - 2 * (I & 3);
    const uint32_t w = *(const uint8_t*)(lds + A + (I >> 2) * Geo<KIND, N>::NS * 64);
    const uint32_t d0 = (uint32_t)((int32_t)(w << (31 - b)) >> 31);
    const uint32_t d1 = (uint32_t)((int32_t)(w << (30 - b)) >> 31);
    A = (A & ~m) | (d0 & m);
    A = (A & ~sh) | (d1 & sh);
    D = (D << 2) | ((w >> b) & 3u);
  } else {
    // I: iteration of the round; group I >> 3 of the staged words
    constexpr int k = I & 7;
    const uint32_t w = *(const uint8_t*)(lds + A + (I >> 3) * Geo<KIND, N>::NS * 128 + 2 * (k & 1));
    const uint32_t t = (w >> (2 * (k >> 1))) & 3u;  // 3 - digit
    A = (A & ~m) | (m & ~(t << sh));
    D = (D << 2) | t;
  }
}

// Steps I .. 0 of a round; phase of step I: (I mod NP) relative to the round.
template <int KIND, int N, int I>
__device__ __forceinline__ void steps(const char* lds, uint32_t& A,
                                      const uint32_t (&m)[Geo<KIND, N>::NP],
                                      const uint32_t (&sh)[Geo<KIND, N>::NP], uint32_t& D) {
  if constexpr (I >= 0) {
    constexpr int P = I % Geo<KIND, N>::NP;
    step<KIND, N, I>(lds, A, m[P], sh[P], D);
    steps<KIND, N, I - 1>(lds, A, m, sh, D);
  }
}

}  // namespace tb

// table: per wavefront (first, count | log2 lanes per item << 16); entries
// count items, or for packed pairs frame pairs, whose (first item, count)
// list follows the wavefronts' entries.
template <int KIND, int N>
__global__ __launch_bounds__(64) void k_tb_rot(const Item* __restrict__ items,
                                               const int2* __restrict__ table, int n_waves,
                                               const uint64_t* __restrict__ surv,
                                               const int32_t* __restrict__ item_end,
                                               uint32_t* __restrict__ bits, int warm) {
  using namespace tb;
  using G = Geo<KIND, N>;
  constexpr int RS = G::RS, RPB = G::RPB, NP = G::NP;
  constexpr bool kPair = KIND == kPairs;
  __shared__ __align__(16) char lds[2 * G::BUF];
  const int lane = threadIdx.x;
  const int h = kPair ? lane >> 5 : 0;
  const int slot = kPair ? lane & 31 : lane;  // (item or pair, segment) of this lane
  const int2 entry = table[blockIdx.x];
  const int first = entry.x, count = entry.y & 0xFFFF, log2g = entry.y >> 16;
  const int g = slot & ((1 << log2g) - 1);
  const int m_idx = slot >> log2g;
  bool have = m_idx < count;
  int ii = first + (have ? m_idx : 0);
  if (kPair) {
    const int2 pr = table[n_waves + ii];
    ii = pr.x + (h < pr.y ? h : 0);
    have = have && h < pr.y;  // a pair of one frame: the second lane idles along
  }
  const Item it = items[ii];
  const int lead = G::STEP == 2 ? it.n_stages & 1 : 0;
  const int Se = it.n_stages - lead;  // stages chased (radix 4: whole iterations)
  const int n = it.n_out;
  const int ob = it.out_begin - lead;  // -1: stage 0 of an odd count is emitted
  const uint32_t* sv = (const uint32_t*)(surv + it.surv_off);
  uint32_t* out = bits + (it.bit_off >> 5);
  // blocks of 32 stages bb .. b_last hold the emitted bits; output word k is
  // (E_{bb+k+1} : E_{bb+k}) >> r.  Lane g owns LB of them.
  const int bb = ob >> 5, r = ob & 31;
  const int n_blk = n > 0 ? ((ob + n - 1) >> 5) - bb + 1 : 0;
  const int n_words = (n + 31) >> 5;
  const int LB = max(1, (n_blk + (1 << log2g) - 1) >> log2g);
  const int b0 = bb + g * LB;
  const int b1 = min(b0 + LB, bb + n_blk);
  const bool active = m_idx < count && b0 < b1;
  const bool last = b1 == bb + n_blk;
  const bool exact = active && (last || b1 + warm >= (Se >> 5) + ((Se & 31) != 0));

  // start of the first chase: time t_top, state s_top there
  int t_top = exact ? Se : 32 * (b1 + warm);
  int s_top = exact ? item_end[it.slot] : 0;
  const uint32_t lane_base = (uint32_t)(slot * 16 + (kPair ? h : 0));
  const uint32_t state_bits = (uint32_t)G::off(G::NS - 1);
  const int r_end = max(b0, 0) * RPB;  // last round of this lane
  uint32_t X = 0, Y = 0, E_low = 0, E_top = 0;
  bool run = active;
  for (int pass = 0;; ++pass) {
    WordGroup wg;
    uint32_t A = lane_base + (uint32_t)G::off(rotl_n(s_top, t_top % N, N));
    // decisions above t_top: the bits of the state there
    const int bt = (t_top - 1) >> 5;  // -1 at time 0
    const uint64_t V = (uint64_t)(uint32_t)s_top << (t_top - 32 * bt);
    uint32_t D = (uint32_t)V, D_up = (uint32_t)(V >> 32), E_up = 0;
    const int r_top = (t_top + RS - 1) / RS - 1;
    const int nr = run ? r_top - r_end + 1 : 0;
    // address bit (packed: digit) of each phase, relative to the round
    uint32_t m[NP], sh[NP];
    {
      const int ph = (max(r_top, 0) * (RS % N)) % N;  // (r_top * RS) mod N
#pragma unroll
      for (int k = 0; k < NP; ++k) {
        const int q = (ph + k * G::STEP) % N;
        sh[k] = (uint32_t)G::bit(q);
        m[k] = (kPair ? 3u : 1u) << sh[k];
        if (KIND == kDigits) sh[k] = 1u << G::bit((q + 1) % N);
      }
    }
    if (run && (t_top & 31) == 0 && (t_top >> 5) == b1) Y = A & state_bits;
    auto fetch = [&](int rd, int k) {
      const uint32_t* src = sv + (int64_t)rd * G::WPR + (kPair ? 4 * h : 0);
      char* dst = lds + (k & 1) * G::BUF;
#pragma unroll
      for (int c = 0; c < G::CH; ++c)
        __builtin_amdgcn_global_load_lds((const void*)(src + (kPair ? 8 : 4) * c),
                                         (lds_ptr_t)(dst + c * 1024), 16, 0, 0);
    };
    // block b is complete in D: its message bits
    auto block_done = [&](int b) {
      const uint32_t E = (uint32_t)(((((uint64_t)D_up) << 32) | D) >> N);
      if (b < b1) {
        const int k = b - bb;
        if (b == b1 - 1 && r != 0) {
          E_top = E;  // needs the bits of the block above: once those are final
        } else if (have && k < n_words) {
          uint32_t w = (uint32_t)(((((uint64_t)E_up) << 32) | E) >> r);
          if (k == n_words - 1 && (n & 31)) w &= (1u << (n & 31)) - 1u;
          wg.put(out, k, w);
        }
      }
      E_up = E;
      D_up = D;
      D = 0;
    };
    if (nr > 0) fetch(r_top, 0);
    for (int k = 0;; ++k) {
      if (__ballot(k < nr) == 0) break;
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      const int rd = r_top - k;
      if (k + 1 < nr) fetch(rd - 1, k + 1);
      if (k < nr) {
        uint32_t d = 0;
        const int lim = t_top - rd * RS;  // stages of this round below t_top
        if (lim >= RS) {
          steps<KIND, N, RS / G::STEP - 1>(lds, A, m, sh, d);
          d = kPair ? ~d : KIND == kDigits ? d : 0u - d;
        } else {
          // the item's last, partial round
#pragma unroll 1
          for (int i = lim / G::STEP - 1; i >= 0; --i) {
            const uint32_t q = (uint32_t)G::bit((rd * RS + i * G::STEP) % N);
            if constexpr (KIND == kWords) {
              const uint32_t x = (*(const uint32_t*)(lds + A) >> (31 - i)) & 1u;
              A = (A & ~(1u << q)) | (x << q);
              d |= x << i;
            } else if constexpr (KIND == kBytes) {
              const uint32_t x =
                  ((uint32_t) * (const uint8_t*)(lds + A + (i >> 3) * G::NS * 64) >> (7 - (i & 7))) & 1u;
              A = (A & ~(1u << q)) | (x << q);
              d |= x << i;
            } else if constexpr (KIND == kDigits) {
              const uint32_t q1 = (uint32_t)G::bit((rd * RS + i * 2 + 1) % N);
              const uint32_t x =
                  ((uint32_t) * (const uint8_t*)(lds + A + (i >> 2) * G::NS * 64) >> (6 - 2 * (i & 3))) & 3u;
              A = (A & ~(1u << q) & ~(1u << q1)) | ((x & 1) << q) | ((x >> 1) << q1);
              d |= x << (2 * i);
            } else {
              const uint32_t w = *(const uint8_t*)(lds + A + (i >> 3) * G::NS * 128 + 2 * (i & 1));
              const uint32_t x = 3u - ((w >> (2 * ((i & 7) >> 1))) & 3u);
              A = (A & ~(3u << q)) | (x << q);
              d |= x << (2 * i);
            }
          }
        }
        // (a whole round of 32 stages has no bits above it in D)
        if constexpr (RS < 32) {
          d &= (1u << (lim < RS ? lim : RS)) - 1u;
          D |= d << ((rd % RPB) * RS);
        } else {
          D |= d;
        }
        if (rd % RPB == 0) {
          const int b = rd / RPB;
          block_done(b);
          if (b == b1) Y = A & state_bits;  // the position at time 32 b1 (buffer bit not in it)
        }
        // the next round's buffer, and its phases
        A ^= (uint32_t)G::BUF;
        constexpr int S = (RS / G::STEP) % NP;  // the phase index moves by -S per round
        if constexpr (S != 0) {
          uint32_t m2[NP], s2[NP];
#pragma unroll
          for (int x = 0; x < NP; ++x) {
            m2[x] = m[(x + NP - S) % NP];
            s2[x] = sh[(x + NP - S) % NP];
          }
#pragma unroll
          for (int x = 0; x < NP; ++x) {
            m[x] = m2[x];
            sh[x] = s2[x];
          }
        }
      }
    }
    if (run) {
      X = A & state_bits;
      if (b0 < 0) block_done(-1);  // the bit below the first whole iteration
      E_low = E_up;
      wg.flush();
    }
    // lane g is right when its state at its upper boundary equals the state
    // lane g+1 reached there
    const uint32_t x_up = (uint32_t)__shfl_down((int)X, 1);
    bool bad = active && !exact && !last && Y != x_up;
    if (__ballot(bad) == 0 || pass > (1 << log2g)) break;
    run = bad;
    if (kPair) {
      // both lanes of a slot stage its words; the one that was right repeats
      const int other = __shfl_xor((int)bad, 32);
      run = active && (bad || other != 0);
    }
    t_top = 32 * b1;
    s_top = rotl_n(G::pos((int)(bad ? x_up : Y)), (N - t_top % N) % N, N);
  }
  // top words that straddle two lanes' blocks
  const uint32_t E_above = (uint32_t)__shfl_down((int)E_low, 1);
  if (active && have && r != 0) {
    const int k = b1 - 1 - bb;
    if (k < n_words) {
      uint32_t w = (uint32_t)(((((uint64_t)(last ? 0u : E_above)) << 32) | E_top) >> r);
      if (k == n_words - 1 && (n & 31)) w &= (1u << (n & 31)) - 1u;
      out[k] = w;
    }
  }
}

// kind_k: 16 * kind (kTb*) + K; table as for k_tb_rot.  (The name and the
// argument list are those of the packed-pair launcher it grew from, which the
// CPU builds of the host code stand in for.)
hipError_t launch_tb_r4p(int kind_k, const Item* items, const int2* table, int n_waves,
                         const uint64_t* surv, const int32_t* item_end, uint32_t* bits, int warm,
                         hipStream_t st) {
  if (n_waves <= 0) return hipSuccess;
#define MV_TB(KIND, N)                                                                       \
  hipLaunchKernelGGL((k_tb_rot<KIND, N>), dim3(n_waves), dim3(64), 0, st, items, table,      \
                     n_waves, surv, item_end, bits, warm);                                   \
  return hipGetLastError()
  switch (kind_k) {
    case tb::kWords * 16 + 3: MV_TB(tb::kWords, 2);
    case tb::kWords * 16 + 4: MV_TB(tb::kWords, 3);
    case tb::kWords * 16 + 5: MV_TB(tb::kWords, 4);
    case tb::kWords * 16 + 6: MV_TB(tb::kWords, 5);
    case tb::kWords * 16 + 7: MV_TB(tb::kWords, 6);
    case tb::kBytes * 16 + 8: MV_TB(tb::kBytes, 7);
    case tb::kBytes * 16 + 9: MV_TB(tb::kBytes, 8);
    case tb::kDigits * 16 + 8: MV_TB(tb::kDigits, 7);
    case tb::kDigits * 16 + 9: MV_TB(tb::kDigits, 8);
    case tb::kPairs * 16 + 5: MV_TB(tb::kPairs, 4);
    case tb::kPairs * 16 + 7: MV_TB(tb::kPairs, 6);
    default: return hipErrorInvalidValue;
  }
#undef MV_TB
}

}  // namespace mivit

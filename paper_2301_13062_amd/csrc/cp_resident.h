// cp_resident.h -- the register-resident rollout loop shared by the
// random-action kernel and the MLP-policy kernel.  Internal to the library.
//
// One lane owns one environment for all T steps; its state never leaves
// VGPRs.  Per step: the action (from the policy functor), dynamics,
// termination; on termination the lane swaps in the start state of its next
// episode, drawn ahead of time.  After every kRefill steps at most the lanes
// that used theirs go on to the next one they hold (up to three, without a
// trajectory), and where a lane has none left the wave or the block draws.
#pragma once

#include <type_traits>
#include <utility>

#include "cp_launch.h"
#include "cp_precision.h"
#include "cp_rows.h"

namespace cp {

constexpr int kResidentBlock = 256;
constexpr int kResidentWaves = kResidentBlock / 64;

// Refill period of the prefetched reset states: no episode started from the
// reset distribution ends before its kRefill-th step, so between two refills
// at most kRefill steps apart a lane ends at most one episode and its
// prefetched start state is always there.
constexpr uint32_t kRefill = 8u;

// Largest |theta| that `steps` steps from the reset distribution (every
// variable within 0.05) can reach: every term of the angular acceleration
// taken with the sign and size that grow it (sin x <= x, |cos| <= 1, the
// divisor at its smallest, at cos = 1) and one percent added to each step
// for rounding in any of the precisions.
constexpr double largest_angle(uint32_t steps) {
  const double g = 9.8, mp = 0.1, m = 1.1, l = 0.5, tau = 0.02;
  double th = 0.05, thd = 0.05;
  for (uint32_t k = 0; k < steps; ++k) {
    const double temp = (10.0 + mp * l * thd * thd * th) / m;
    const double acc = (g * th + temp) / (l * (4.0 / 3.0 - mp / m));
    const double th1 = th + tau * thd;
    thd = 1.01 * (thd + tau * acc);
    th = 1.01 * th1;
  }
  return th;
}
// (x, from 0.05 at 0.05 per second and below 12 per second^2, stays far
// inside 2.4 meanwhile)
static_assert(largest_angle(kRefill - 1u) < 0.2094, "an episode may end within a refill period");

__device__ __forceinline__ unsigned long long wave_sum_u64(unsigned long long v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    const uint32_t lo = __shfl_xor(uint32_t(v), off, 64);
    const uint32_t hi = __shfl_xor(uint32_t(v >> 32), off, 64);
    v += (static_cast<unsigned long long>(hi) << 32) | lo;
  }
  return v;
}

// Adds a block's sums to global[0], global[1] with one atomic instruction:
// every wave adds its lanes' sums to the block's in LDS and counts itself, the
// wave that counts last publishes them (lanes 0 and 1 one sum each).  No
// barrier: waves end at different times, and ended ones leave their issue
// slots to the others, where waves waiting at a barrier slowed the rest
// (1,048,576 x 1,000 in binary16 1,375 -> 1,250 us).
// Atomics on one line come back at about 10 ns each however many blocks
// issue them (65,536 blocks adding their two sums one after the other cost
// a 230 us launch another 1.34 ms), so kernels whose blocks are short call it
// from a bounded grid.
template <int kBlockThreads>
struct BlockTotals {
  unsigned long long sums[2];
  uint32_t waves;

  // Before a barrier that every wave passes.
  __device__ __forceinline__ void clear() {
    if (threadIdx.x == 0u) {
      sums[0] = sums[1] = 0u;
      waves = 0u;
    }
  }

  // Called once by every lane of every wave.
  __device__ __forceinline__ void publish(unsigned long long *global, unsigned long long a,
                                          unsigned long long b) {
    a = wave_sum_u64(a);
    b = wave_sum_u64(b);
    const uint32_t lane = threadIdx.x & 63u;
    uint32_t before = 0u;
    if (lane < 2u) atomicAdd(&sums[lane], lane == 0u ? a : b);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    if (lane == 0u) before = atomicAdd(&waves, 1u);
    before = __builtin_amdgcn_readfirstlane(before);
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    if (before + 1u == uint32_t(kBlockThreads / 64) && lane < 2u) {
      const unsigned long long t = atomicAdd(&sums[lane], 0ull);
      if (t) atomicAdd(&global[lane], t);
    }
  }
};

// The value of lane (this lane ^ kMask), within rows of 16 lanes.
template <int kMask>
__device__ __forceinline__ uint32_t lane_xor(uint32_t v) {
  const int x = int(v);
  if (kMask == 1) return uint32_t(__builtin_amdgcn_mov_dpp(x, 0xB1, 0xF, 0xF, true));  // quad_perm 1,0,3,2
  if (kMask == 2) return uint32_t(__builtin_amdgcn_mov_dpp(x, 0x4E, 0xF, 0xF, true));  // quad_perm 2,3,0,1
  if (kMask == 8) return uint32_t(__builtin_amdgcn_mov_dpp(x, 0x128, 0xF, 0xF, true));  // row_ror:8
  static_assert(kMask == 1 || kMask == 2 || kMask == 4 || kMask == 8, "a bit of a row's lane");
  const int m = __builtin_amdgcn_mov_dpp(x, 0x141, 0xF, 0xF, true);  // row_half_mirror: ^ 7
  return uint32_t(__builtin_amdgcn_mov_dpp(m, 0x1B, 0xF, 0xF, true));  // quad_perm 3,2,1,0: ^ 3
}

// One stage of the transposition below: bits whose index has bit kS set (or
// clear, in a lane with that bit) come from the lane ^ kS.
template <int kS>
__device__ __forceinline__ uint32_t transpose_stage(uint32_t x, uint32_t lane) {
  constexpr uint32_t kLow = kS == 8 ? 0x00FF00FFu : kS == 4 ? 0x0F0F0F0Fu : kS == 2 ? 0x33333333u : 0x55555555u;
  const bool high = (lane & uint32_t(kS)) != 0u;
  const uint32_t keep = high ? ~kLow : kLow, y = lane_xor<kS>(x);
  const uint32_t r = __builtin_amdgcn_alignbit(y, y, high ? kS : 32 - kS);
  return (x & keep) | (r & ~keep);
}

// The 64 x 64 bit matrix whose row L is lane L's (a, b), a the columns 0 to
// 31, transposed: bit i of lane L's a' is row i's column L, of b' row i + 32's.
__device__ __forceinline__ void transpose64(uint32_t &a, uint32_t &b) {
  const uint32_t lane = threadIdx.x & 63u;
  auto s32 = __builtin_amdgcn_permlane32_swap(a, b, false, false);
  a = s32[0];
  b = s32[1];
  auto half = [&](uint32_t x) {
    // even rows of 16 lanes: both rows' low halves; odd ones: the high halves
    auto s16 = __builtin_amdgcn_permlane16_swap(x, x, false, false);
    x = __builtin_amdgcn_perm(s16[1], s16[0], (lane & 16u) ? 0x07060302u : 0x05040100u);
    x = transpose_stage<8>(x, lane);
    x = transpose_stage<4>(x, lane);
    x = transpose_stage<2>(x, lane);
    return transpose_stage<1>(x, lane);
  };
  a = half(a);
  b = half(b);
}

// The groups of steps of a launch (resident_rollout).
enum class Group { kFirst, kRound, kRest };

// Random actions.  The actions of a 64-environment block at one step are one
// generator output (see action_bit).  Every 64 steps each lane computes the
// wave's output of one of the next 64 steps, and the wave transposes them, so
// that each lane holds its environment's actions of these steps as two words,
// the first step in the top bit: a step's action is the word's top bit and a
// shift (two full-rate instructions, where reading the step's output from the
// owning lane and selecting by it took five at half rate).  Waves start at
// multiples of 64 environments after the launch's first one, so either every
// wave is aligned to a block (kAligned: the launch starts at a multiple of 64)
// or every wave straddles two blocks and computes both.  A launch of at most
// kFew steps, one group without a refill, selects by the outputs themselves:
// there the transposition costs more than it saves (1,048,576 environments
// without outputs, of one step 10.9 -> 9.7 us, of two 12.1 -> 10.4, of five 13.9
// -> 13.3; of eight 16.5 and 16.9).
template <bool kAligned>
struct HashPolicy {
  static constexpr bool kUnrolled = true;      // the rounds of kRefill steps
  static constexpr bool kBlockRefill = true;   // refills of the trajectory form
  static constexpr bool kAhead = true;         // more than one start state ahead
  static constexpr uint32_t kEnvsPerWave = 64;
  U2 key;
  uint32_t g0, off;  // the wave's first block and place in it
  uint32_t word, later;  // this lane's actions from the next step on; of steps 32 .. 63
  uint32_t few;          // the steps of a launch of at most kFew, else 0
  static constexpr uint32_t kFew = kRefill;

  __device__ __forceinline__ HashPolicy(U2 k, uint32_t env, uint32_t T) : key(k), few(T <= kFew ? T : 0u) {
    const uint32_t first = uint32_t(__builtin_amdgcn_readfirstlane(int(env)));
    g0 = first >> 6;
    off = first & 63u;
  }

  // The wave's output of a step: bit i the action of its i-th environment.
  __device__ __forceinline__ U2 output(uint32_t step) const {
    const U2 w = threefry2x32(key.a, key.b, g0, step);
    if (kAligned) return w;
    const U2 w1 = threefry2x32(key.a, key.b, g0 + 1u, step);
    const unsigned long long lo = (static_cast<unsigned long long>(w.b) << 32) | w.a;
    const unsigned long long hi = (static_cast<unsigned long long>(w1.b) << 32) | w1.a;
    const unsigned long long both = off == 0u ? lo : (lo >> off) | (hi << (64u - off));
    return U2{uint32_t(both), uint32_t(both >> 32)};
  }

  // Called before a group of steps, with its first step: the launch's first
  // (kFirst) or a multiple of kRefill, of a full round (kRound) or not (kRest).
  // A launch of at most kFew steps has no full round.
  template <Group kGroup>
  __device__ __forceinline__ void prepare(uint32_t t) {
    if (kGroup != Group::kRound && few != 0u) {
      if (kGroup == Group::kRest) return;
      const U2 w = output(t + (threadIdx.x & (kFew - 1u)));
      word = 0u;
#pragma unroll 1
      for (int k = 0; k < int(few); ++k) {
        const uint32_t a = uint32_t(__builtin_amdgcn_readlane(int(w.a), k));
        const uint32_t b = uint32_t(__builtin_amdgcn_readlane(int(w.b), k));
        if (__builtin_amdgcn_inverse_ballot_w64((static_cast<unsigned long long>(b) << 32) | a))
          word |= 0x80000000u >> k;
      }
      return;
    }
    if (kGroup != Group::kFirst && (t & 31u) != 0u) return;
    if (kGroup != Group::kFirst && (t & 63u) != 0u) {
      word = later;
      return;
    }
    // rows in descending order of their steps within each half
    U2 w = output((t & ~63u) + ((threadIdx.x & 63u) ^ 31u));
    transpose64(w.a, w.b);
    later = w.b;
    word = (t & 32u) ? w.b : w.a;
    if (kGroup == Group::kFirst) word <<= t & 31u;
  }

  // The action of the next step in the top bit.
  template <class St>
  __device__ __forceinline__ uint32_t operator()(const St &) {
    const uint32_t w = word;
    word <<= 1;
    return w;
  }
};

// What a launch stores per step: nothing, whichever of obs [T][4][n] (in the
// state's type), reward [T][n] f32 and done [T][n] u8 are given, or all three
// with every byte offset within a plane below 2^32 (no tests in the loop), each
// wave its own environments (kAll) or the block its piece of a row (kRows).
enum class Traj { kNone, kAny, kAll, kRows };

// The kernel without tests in the loop (kAll) leaves three waves per SIMD in
// binary32 and two in binary64, the other one (kAny) seven and five.  Fewer waves
// store nearer to each other (4,194,304 x 5 in binary32: 124 us, kAny 135; x 32:
// 605 and 625) and tests cost small batches (4,096 x 64: 21 us, kAny 27), but a
// launch of few steps lacks the waves that cover its loads: one step of
// 1,048,576 environments 14.1 and 12.5 us, two of 4,194,304 76 and 65 (binary64,
// one step of 4,194,304: 119 and 92, two of 1,048,576 29.6 and 28.3).
constexpr uint32_t kAllMinSteps = 4u;

inline Traj traj_kind(const RolloutParams &p, size_t elem) {
  if (!p.obs && !p.reward && !p.done) return Traj::kNone;
  const bool off32 = uint64_t(p.n) * (elem > 4 ? elem : 4) <= (uint64_t(1) << 32);
  return p.obs && p.reward && p.done && off32 ? Traj::kAll : Traj::kAny;
}

// Threads per block of a launch that stores by rows (kRows, cp_rows.h), or 0.
inline uint32_t rows_block(const RolloutParams &p, size_t elem) {
  if (traj_kind(p, elem) != Traj::kAll) return 0u;
  return rows_block(p.n, p.T, uint32_t(elem), reinterpret_cast<uintptr_t>(p.obs),
                    reinterpret_cast<uintptr_t>(p.reward));
}

// Whether a launch has trajectory rows off the 128-byte lines
// (RolloutParams::ragged).
inline bool rows_ragged(const RolloutParams &p, size_t elem) {
  return traj_kind(p, elem) != Traj::kNone &&
         !rows_on_lines(p.n, uint32_t(elem), reinterpret_cast<uintptr_t>(p.obs),
                        reinterpret_cast<uintptr_t>(p.reward));
}

// Stores of one step (obs, reward and done: the step's rows).  Each plane's
// base is wave-uniform (scalar arithmetic); kOff32 takes the scalar-base form
// with the lane's fixed 32-bit offset, otherwise 64-bit vector addresses.
// Plain (write-back) stores: the waves of a launch are at different steps at
// any moment, so each writes its pieces of many planes far apart, and
// non-temporal stores of those pieces measured 10-15% slower (7.2 against
// 6.2-6.5 ms for 16,777,216 x 100) than stores the L2 merges into whole lines
// first.
template <bool kAll, bool kOff32, class T, class S>
__device__ __forceinline__ void store_traj(T *obs, float *reward, uint8_t *done, uint32_t n,
                                           uint32_t i, const S &s, bool d) {
  if (kAll || obs) {
    *elem<kOff32>(obs, i) = s.x;
    *elem<kOff32>(obs + n, i) = s.xd;
    *elem<kOff32>(obs + 2u * size_t(n), i) = s.th;
    *elem<kOff32>(obs + 3u * size_t(n), i) = s.thd;
  }
  if (kAll || reward) *elem<kOff32>(reward, i) = 1.0f;
  if (kAll || done) *elem<kOff32>(done, i) = uint8_t(d);
}

// On the lanes of `m` (wave-uniform): s = nxt, and lr = r.  Written as moves
// under the mask: a move issues at twice the rate of a select, and selects
// one after the other on the same condition at a fraction of it (measured:
// 4.3 moves, 2.3 selects on a scalar mask, 0.4 successive selects on vcc per
// CU and ns).  r: an integral_constant or a wave-uniform number.
#define CP_TAKE(mov, r_constraint, r_value)                                                       \
  unsigned long long saved;                                                                       \
  asm volatile(                                                                                   \
      "s_and_saveexec_b64 %[sv], %[m]\n\t" mov " %[x], %[nx]\n\t" mov " %[xd], %[nxd]\n\t" mov     \
      " %[th], %[nth]\n\t" mov " %[thd], %[nthd]\n\tv_mov_b32 %[lr], %[r]\n\ts_mov_b64 exec, %[sv]" \
      : [x] "+v"(s.x), [xd] "+v"(s.xd), [th] "+v"(s.th), [thd] "+v"(s.thd), [lr] "+v"(lr),        \
        [sv] "=&s"(saved)                                                                         \
      : [m] "s"(m), [nx] "v"(nxt.x), [nxd] "v"(nxt.xd), [nth] "v"(nxt.th), [nthd] "v"(nxt.thd),   \
        [r] r_constraint(r_value)                                                                 \
      : "scc")

template <int r>
__device__ __forceinline__ void take(unsigned long long m, State &s, const State &nxt,
                                     uint32_t &lr, std::integral_constant<int, r>) {
  CP_TAKE("v_mov_b32", "i", r);
}
__device__ __forceinline__ void take(unsigned long long m, State &s, const State &nxt,
                                     uint32_t &lr, uint32_t r) {
  CP_TAKE("v_mov_b32", "s", r);
}
template <int r>
__device__ __forceinline__ void take(unsigned long long m, State64 &s, const State64 &nxt,
                                     uint32_t &lr, std::integral_constant<int, r>) {
  CP_TAKE("v_mov_b64", "i", r);
}
__device__ __forceinline__ void take(unsigned long long m, State64 &s, const State64 &nxt,
                                     uint32_t &lr, uint32_t r) {
  CP_TAKE("v_mov_b64", "s", r);
}
#undef CP_TAKE
__device__ __forceinline__ void take(unsigned long long m, State16 &s, const State16 &nxt,
                                     uint32_t &lr, uint32_t r) {
  if (__builtin_amdgcn_inverse_ballot_w64(m)) {
    s = nxt;
    lr = r;
  }
}

// On the lanes of m: dst = src.
__device__ __forceinline__ void move_on(unsigned long long m, State &dst, const State &src) {
  unsigned long long saved;
  asm volatile(
      "s_and_saveexec_b64 %[sv], %[m]\n\tv_mov_b32 %[x], %[nx]\n\tv_mov_b32 %[xd], %[nxd]\n\t"
      "v_mov_b32 %[th], %[nth]\n\tv_mov_b32 %[thd], %[nthd]\n\ts_mov_b64 exec, %[sv]"
      : [x] "+v"(dst.x), [xd] "+v"(dst.xd), [th] "+v"(dst.th), [thd] "+v"(dst.thd), [sv] "=&s"(saved)
      : [m] "s"(m), [nx] "v"(src.x), [nxd] "v"(src.xd), [nth] "v"(src.th), [nthd] "v"(src.thd)
      : "scc");
}
template <class S>
__device__ __forceinline__ void move_on(unsigned long long m, S &dst, const S &src) {
  if (__builtin_amdgcn_inverse_ballot_w64(m)) dst = src;
}

// f(integral_constant 0), ..., f(integral_constant kCount - 1)
template <class F, int... r>
__device__ __forceinline__ void each_of(F &f, std::integer_sequence<int, r...>) {
  (f(std::integral_constant<int, r>{}), ...);
}

// p, the same in every lane, as a scalar.
template <class T>
__device__ __forceinline__ T *wave_uniform(T *p) {
  const uintptr_t v = reinterpret_cast<uintptr_t>(p);
  const uint32_t lo = uint32_t(__builtin_amdgcn_readfirstlane(int(uint32_t(v))));
  const uint32_t hi = uint32_t(__builtin_amdgcn_readfirstlane(int(uint32_t(v >> 32))));
  return reinterpret_cast<T *>(uintptr_t(hi) << 32 | lo);
}

// The lane's environment of a launch: kEnvsPerWave consecutive ones per wave;
// with fewer than 64 the lanes past them run the first ones' again (the same
// values) and store nothing.
template <class Policy>
__device__ __forceinline__ uint32_t lane_env(uint32_t block) {
  constexpr uint32_t kEnvs = Policy::kEnvsPerWave;
  return (block * kResidentWaves + (threadIdx.x >> 6)) * kEnvs + (threadIdx.x & (kEnvs - 1u));
}

// The block's place in the batch, blocks of one XCD (every eighth is launched
// on the same one) next to each other: for trajectories whose rows do not start
// on 128-byte lines (random actions; 50,001 x 952 in binary32 328 us as
// launched, 266 so, 150,001 x 317 353 and 291, 1,000,003 x 47 339 and 290; with
// aligned rows 4,194,240 x 64 1,201 and 1,137, but 4,194,304 x 64 1,118 and
// 1,130, 16,777,216 x 20 1,509 and 1,606).
__device__ __forceinline__ uint32_t xcd_block() {
  const uint32_t x = blockIdx.x & 7u, q = gridDim.x >> 3, r = gridDim.x & 7u;
  return x * q + (x < r ? x : r) + (blockIdx.x >> 3);
}

// Whole rows by block (kRows), for trajectories whose rows do not all start on
// a 128-byte line.  Waves that store their own 64 values each then leave parts
// of two lines, completed by another wave at another time -- mostly after
// the part was written out, which costs a multiple of a whole line.  So
// the block puts a step's values into LDS and stores its piece of each row
// from the row's own first line boundary on (`turned`): all lines but the two
// at the piece's ends are written whole by one instruction, and the blocks
// of one XCD lie next to each other, so that most end lines too are completed
// in the same L2.  4,194,303 x 64 in binary32: 2,127 us stored by waves,
// 1,700 by blocks of 256 on consecutive places, 1,850 by blocks of 1,024 as
// launched, 1,196 by those on consecutive places (aligned rows: 1,109); in
// binary64 3,258 -> 1,949.
template <class T, int kEnvs>
struct RowStage {
  T v[4][kEnvs];
  uint8_t done[kEnvs];
};

// The lane's element of the block's piece of a row: the elements from the
// first 128-byte line on come first, those before it last.
template <int kEnvs>
__device__ __forceinline__ uint32_t turned(const void *piece, uint32_t elem_bytes, uint32_t at = 0u) {
  const uint32_t head = (0u - uint32_t(reinterpret_cast<uintptr_t>(piece))) & 127u;
  return (threadIdx.x + at + head / elem_bytes) & uint32_t(kEnvs - 1);
}

// The loop.  `policy(s)` returns, in the top bit, the action of the next step
// for the lane's pre-step state s; it is called by every lane of the wave at
// every step (policies may use cross-lane operations).  P is the precision of the
// state, the step and the obs trajectory (the state and obs pointers of p
// point at P::T values).
//
// What bounds it is vector issue (the trajectory form: its stores), so the
// step is kept to the arithmetic, two compares, the action's bit and shift
// and five moves: the episode length is not counted (the step of the
// latest termination is kept instead), the episode index is brought up to
// date at the refills only, and rounds start at multiples of kRefill of the
// global step, so that the generator test runs once per round.  Measured with
// the divisions' cheaper forms against the earlier loop (length counted,
// selects, a second termination tested for at every step): 1,048,576 x 1,000
// in binary32 1.293 -> 1.227 ms, in binary64 2.54 -> 2.04 ms; 1,024 x 200,
// where a step costs one wave's instruction stream, 41.8 -> 33.4 us.  With
// the actions held per lane, a ballot per compare and more than one start state
// ahead: 0.92 and 1.85 ms, 29.2 us.
//
// block: the block's place in the batch.
template <Traj kTraj, class Policy, class P = PrecF32, int kBlockThreads = kResidentBlock>
__device__ __forceinline__ void resident_rollout(const RolloutParams &p, Policy &policy, uint32_t block) {
  using T = typename P::T;
  using S = typename P::S;
  constexpr int kWaves = kBlockThreads / 64;
  __shared__ BlockTotals<kBlockThreads> totals;
  if (p.global) {
    totals.clear();
    __syncthreads();
  }
  T *const px = reinterpret_cast<T *>(p.x);
  T *const pxd = reinterpret_cast<T *>(p.xd);
  T *const pth = reinterpret_cast<T *>(p.th);
  T *const pthd = reinterpret_cast<T *>(p.thd);
  const uint32_t piece0 = block * uint32_t(kBlockThreads);  // kRows: the block's first one
  const uint32_t i = kTraj == Traj::kRows ? piece0 + threadIdx.x : lane_env<Policy>(block);
  const bool off32 = uint64_t(p.n) * (sizeof(T) > 4 ? sizeof(T) : 4) <= (uint64_t(1) << 32);
  const bool valid = i < p.n, owner = valid && (threadIdx.x & 63u) < Policy::kEnvsPerWave;
  const uint32_t env = p.env_base + i;
  // Lanes past the end run the loop too (the wave stays converged for the
  // cross-lane operations) and store nothing.  They take the first step, which
  // evaluates angles beyond 1/4 and NaN by the library's routines (1 us for the
  // wave), at rest, and the others on a NaN state: it never terminates.
  S s{T(0), T(0), T(0), T(0)};
  uint32_t k0 = 0u, len0 = 0u;
  if (valid) {
    s = S{px[i], pxd[i], pth[i], pthd[i]};
    k0 = p.ep_index[i];
    len0 = p.ep_len[i];
  }
  // The lane is in episode k, or in k + 1 if its bit of `used` is set: it
  // ended an episode since the last refill, at the lr-th step after it, and
  // used the prefetched start state nxt (of episode k + 1).
  uint32_t k = k0, lr = 0u, last = 0u;
  unsigned long long used = 0u;
  S nxt = P::draw(p.krst, env, k + 1u);
  // The start states after it that the lane holds, in order: more[d] (of
  // episode k + 2 + d) on the lanes of held[d].
  constexpr int kMore = kTraj == Traj::kNone && Policy::kAhead ? P::kAhead - 1 : 0;
  S more[kMore + 1];
  unsigned long long held[kMore + 1];
#pragma unroll
  for (int d = 0; d <= kMore; ++d) {
    more[d] = nxt;
    held[d] = 0u;
  }
  // rows of the step's trajectory outputs
  T *row_obs = reinterpret_cast<T *>(p.obs);
  float *row_reward = p.reward;
  uint8_t *row_done = p.done;
  // The block's piece of the step's rows, through LDS (two stages in turn, so
  // that one barrier per step orders a stage's readers before its next
  // writers).
  uint32_t turn = 0u;
  const bool whole = piece0 + uint32_t(kBlockThreads) <= p.n;
  auto store_rows = [&](bool d) {
    __shared__ RowStage<T, kBlockThreads> stages[2];
    RowStage<T, kBlockThreads> &st = stages[turn];
    turn ^= 1u;
    st.v[0][threadIdx.x] = s.x;
    st.v[1][threadIdx.x] = s.xd;
    st.v[2][threadIdx.x] = s.th;
    st.v[3][threadIdx.x] = s.thd;
    st.done[threadIdx.x] = uint8_t(d);
    __syncthreads();
#pragma unroll
    for (uint32_t c = 0; c < 4u; ++c) {
      T *const piece = row_obs + size_t(c) * p.n + piece0;
      const uint32_t e = turned<kBlockThreads>(piece, sizeof(T));
      if (whole || piece0 + e < p.n) *elem<true>(piece, e) = st.v[c][e];
    }
    float *const piece_r = row_reward + piece0;
    const uint32_t er = turned<kBlockThreads>(piece_r, sizeof(float));
    if (whole || piece0 + er < p.n) *elem<true>(piece_r, er) = 1.0f;
    uint8_t *const piece_d = row_done + piece0;
    const uint32_t ed = turned<kBlockThreads>(piece_d, 1u);
    if (whole || piece0 + ed < p.n) *elem<true>(piece_d, ed) = st.done[ed];
  };
  // One step, the r-th after the last refill; `limited`:
  // the state is one a step produced (every step after a launch's first), its
  // angle within the limit or NaN.
  auto step = [&](auto r, auto limited) {
    S o = P::template step<decltype(limited)::value>(s, policy(s));
    const unsigned long long m = P::template done<Policy::kUnrolled>(o);
    take(m, o, nxt, lr, r);
    used |= m;
    s = o;
    if constexpr (kTraj == Traj::kRows) {
      store_rows(__builtin_amdgcn_inverse_ballot_w64(m));
    } else if constexpr (kTraj != Traj::kNone) {
      const bool d = __builtin_amdgcn_inverse_ballot_w64(m);
      if (owner) {
        if (kTraj == Traj::kAll || off32)
          store_traj<kTraj == Traj::kAll, true>(row_obs, row_reward, row_done, p.n, i, s, d);
        else
          store_traj<false, false>(row_obs, row_reward, row_done, p.n, i, s, d);
      }
    }
    if constexpr (kTraj != Traj::kNone) {
      if (kTraj >= Traj::kAll || row_obs) row_obs += 4u * size_t(p.n);
      if (kTraj >= Traj::kAll || row_reward) row_reward += p.n;
      if (kTraj >= Traj::kAll || row_done) row_done += p.n;
      // In binary16 the rows' addresses in scalar registers: the compiler
      // carries those of kAll in vector ones (187, two waves per SIMD; 112 and
      // four), which in binary32 and binary64 serves long launches (kAllMinSteps).
      // 4,194,304 x 32 from an env_base of 1: 585 -> 457 us, x 2 87 -> 65.
      if constexpr (kTraj == Traj::kAll && sizeof(T) == 2) {
        row_obs = wave_uniform(row_obs);
        row_reward = wave_uniform(row_reward);
        row_done = wave_uniform(row_done);
      }
    }
  };
  // After the steps from the j-th of this launch on: the lanes that ended an
  // episode (about a third of them after kRefill steps) count it.
  auto count = [&](uint32_t j) {
    const bool mine = __builtin_amdgcn_inverse_ballot_w64(used);
    used = 0u;
    if (mine) {
      k += 1u;
      last = j + lr;
    }
    return mine;
  };
  // ... and go on to the next start state they hold.  Where a lane has none
  // left, the wave draws: every lane short of kAhead start states its next.
  // A draw costs as much as two steps and a third of the lanes ends an
  // episode in a round; with three (two) states ahead the wave draws after 47
  // (57) of 100 rounds instead of after each, most of its lanes with use
  // (1,048,576 x 1,000 in binary64 1,904 us with one, 1,852 with two, 1,848
  // with three at a wave per SIMD fewer).
  auto refill_wave = [&](uint32_t j) {
    const unsigned long long u = used;
    if (u == 0u) return;
    if constexpr (kMore == 0) {
      if (count(j)) nxt = P::draw(p.krst, env, k + 1u);
    } else {
      count(j);
      move_on(u, nxt, more[0]);
      const unsigned long long none = u & ~held[0];
#pragma unroll
      for (int d = 0; d < kMore; ++d) {
        if (d + 1 < kMore) move_on(u, more[d], more[d + 1]);
        held[d] = (held[d] & ~u) | (d + 1 < kMore ? held[d + 1] & u : 0u);
      }
      if (none == 0u) return;
      uint32_t episode = k + (__builtin_amdgcn_inverse_ballot_w64(none) ? 1u : 2u);
#pragma unroll
      for (int d = 0; d < kMore - 1; ++d)
        episode += __builtin_amdgcn_inverse_ballot_w64(held[d]) ? 1u : 0u;
      const S drawn = P::draw(p.krst, env, episode);
      move_on(none, nxt, drawn);
      unsigned long long room = ~none;  // lanes whose states before more[d] are there
#pragma unroll
      for (int d = 0; d < kMore; ++d) {
        move_on(room & ~held[d], more[d], drawn);
        const unsigned long long there = held[d];
        held[d] |= room;
        room = there;
      }
    }
  };
  // The same refill served by the block together, for the kernel writing a
  // trajectory (bound by its stores, where fewer vector instructions mean
  // less interference with them: 7.1 -> 6.8 ms at 16,777,216 x 100; the
  // compute-bound kernels lose more in the barriers than they save).  The
  // requests are packed into consecutive slots in LDS (wave counts, then
  // each lane's rank among its wave's requests), thread r draws request r --
  // one generator pass for the block's requests instead of one for every
  // wave with any -- and the requesting lanes read their states back.  Every
  // thread of the block takes part (the loop's trip counts are the block's);
  // the wave counts are double-buffered by round, so that a round's counts
  // are never overwritten while a wave may still read them.
  uint32_t parity = 0u;
  auto refill_block = [&](uint32_t j) {
    __shared__ uint32_t wave_cnt[2][kWaves];
    __shared__ uint32_t req_env[kBlockThreads], req_k[kBlockThreads];
    __shared__ S got[kBlockThreads];
    const uint32_t wave = threadIdx.x >> 6;
    const unsigned long long m = used;
    if ((threadIdx.x & 63u) == 0u) wave_cnt[parity][wave] = uint32_t(__popcll(m));
    __syncthreads();
    uint32_t base = 0u, total = 0u;
#pragma unroll
    for (uint32_t v = 0; v < uint32_t(kWaves); ++v) {
      const uint32_t c = wave_cnt[parity][v];
      base += v < wave ? c : 0u;
      total += c;
    }
    parity ^= 1u;
    if (total == 0u) return;  // the same for the whole block
    const uint32_t slot =
        base + __builtin_amdgcn_mbcnt_hi(uint32_t(m >> 32), __builtin_amdgcn_mbcnt_lo(uint32_t(m), 0u));
    const bool mine = count(j);
    if (mine) {
      req_env[slot] = env;
      req_k[slot] = k + 1u;
    }
    __syncthreads();
    if (threadIdx.x < total) got[threadIdx.x] = P::draw(p.krst, req_env[threadIdx.x], req_k[threadIdx.x]);
    __syncthreads();
    if (mine) nxt = got[slot];
  };
  auto refill = [&](uint32_t j) {
    if constexpr (kTraj != Traj::kNone && Policy::kBlockRefill) refill_block(j);
    else refill_wave(j);
  };
  // Groups of at most kRefill steps: the launch's first step (any state) with
  // single steps up to a multiple of kRefill, rounds of kRefill steps
  // (unrolled), the remaining steps.  An environment that ends its episode at
  // the first step is at most kRefill - 1 steps into the next one when the group
  // ends, so a group needs one start state.  After a group comes a refill, after
  // a last one of single steps only its count: launches of few steps, whose
  // refills would all be for steps that do not come, pay for none (one step of
  // 1,048,576 environments with all outputs, 16.9 -> 14.1 us; asked after every
  // round too, 1,024 x 200 takes 30.4 us instead of 29.0).
  using any_angle = std::integral_constant<bool, false>;
  using limited_angle = std::integral_constant<bool, true>;
  uint32_t j = 0u;  // steps done
  auto singles = [&](uint32_t first, uint32_t end) {  // first: the group's first step
    for (; j < end; ++j) step(j - first, limited_angle{});
    if (j < p.T) refill(first);
    else count(first);
  };
  policy.template prepare<Group::kFirst>(p.t0);
  step(0u, any_angle{});
  j = 1u;
  if (!valid) s.x = s.xd = s.th = s.thd = T(__builtin_nanf(""));
  const uint32_t lead = (0u - (p.t0 + 1u)) & (kRefill - 1u);
  singles(0u, p.T < 1u + lead ? p.T : 1u + lead);
  for (; j + kRefill <= p.T; j += kRefill) {
    policy.template prepare<Group::kRound>(p.t0 + j);
    if constexpr (Policy::kUnrolled && kTraj != Traj::kRows) {
      auto one = [&](auto r) { step(r, limited_angle{}); };
      each_of(one, std::make_integer_sequence<int, int(kRefill)>{});
    } else {
#pragma unroll 1
      for (uint32_t r = 0; r < kRefill; ++r) {
        // A step's code from a multiple of 8 bytes on: most of the MLP's
        // instructions take 8, and from an odd word on its loop takes 2.5%
        // longer (4,194,304 x 500: 75.4 and 77.3 ms).
        if constexpr (!Policy::kUnrolled) asm volatile(".p2align 3");
        step(r, limited_angle{});
      }
    }
    refill(j);
  }
  if (j < p.T) {
    policy.template prepare<Group::kRest>(p.t0 + j);
    singles(j, p.T);
  }
  // Over the rollout an environment's terminations are the growth of its
  // episode index, its episode length counts from its latest termination and
  // its finished returns are T + len(start) - len(end); the summed reward of T
  // steps (1 each, accumulated in binary32) is T up to 2^24, where the
  // binary32 sum stops growing.
  const uint32_t len = k != k0 ? p.T - 1u - last : len0 + p.T;
  const uint32_t n_done = k - k0;
  const uint32_t returns = p.T + len0 - len;
  if (owner) {
    px[i] = s.x;
    pxd[i] = s.xd;
    pth[i] = s.th;
    pthd[i] = s.thd;
    p.ep_index[i] = k;
    p.ep_len[i] = len;
    // A rollout split over several launches adds to what the earlier
    // launches wrote; the reward sum keeps the semantics of adding 1.0f once
    // per step in binary32 (exact up to 2^24, constant from there on).
    if (p.done_count) p.done_count[i] = (p.first ? 0u : p.done_count[i]) + n_done;
    if (p.total_reward) {
      const float prev = p.first ? 0.0f : p.total_reward[i];
      const float cap = float(1u << 24);
      p.total_reward[i] = prev >= cap ? prev : __builtin_fminf(prev + float(p.T), cap);
    }
    if (p.ret_sum) p.ret_sum[i] = (p.first ? 0u : p.ret_sum[i]) + returns;
  }
  if (p.global) totals.publish(p.global, owner ? n_done : 0u, owner ? returns : 0u);
}

}  // namespace cp

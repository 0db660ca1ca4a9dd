// cp_resident16.hip -- the register-resident rollout in binary16 with two
// environments per lane (the binary16 precision of the hand-written CUDA
// port the paper compares against, Sec. "Comparison with CUDA
// implementation"), used when the launch's first environment is a multiple
// of 64.  Results equal the one-environment-per-lane binary16 kernel bit
// for bit (every operation the correctly rounded binary16 operation); only
// the instruction selection differs:
//  * lane L of a wave holds environments base + L and base + 64 + L in the
//    low and high halves of packed registers; additions, subtractions and
//    products of the step are packed binary16 instructions (v_pk_add_f16,
//    v_pk_mul_f16: two values, each rounded once);
//  * sin and cos of an angle up to 1/4 are read from a table of the
//    correctly rounded binary16 values (cp_f16_table.h) staged in LDS, one
//    ds_read_b32 per environment for both;
//  * a / m (the binary16 total mass) is a times 1/m held as two binary16
//    numbers, in two packed operations (div_mass2); at a launch's first step,
//    whose dividends may be any, one mixed-precision multiply-add rounding the
//    exact product a * RN32(1/m) once to binary16: equal to the correctly
//    rounded quotient for every binary16 a, the exact quotients lying at least
//    2^-21 (relative) from a binary16 rounding boundary while RN32(1/m) is
//    within 2^-24 of 1/m;
//  * the angular acceleration num / den is num times RN32(1/den), rounded
//    once the same way: every divisor the step can form is one of 94
//    binary16 values (0.621 .. 0.667), whose reciprocals sit in a second LDS
//    table, and for each of them every binary16 quotient lies at least
//    2^-22.4 (relative) from a rounding boundary, farther than RN32(1/den)
//    is from 1/den (2^-24).  The divisor is a function of the cosine alone,
//    so a step whose cosine comes from the table reads RN32(1/den) from a
//    third table keyed by the cosine (65 values) instead of forming den;
//  * the episode counters are brought up to date at the refills of the
//    prefetched start states only, and the episode length at the end from
//    the step of the latest termination.
// States a step produces hold angles within the 12-degree limit or NaN, so
// only a launch's first step can meet an angle beyond the table: it is
// peeled off the loop, and the loop's steps read the table alone (NaN
// angles reading entries of NaNs).
// The actions of a wave's 128 environments are two 64-environment blocks of
// the random stream, transposed every 64 steps so that a lane holds its own.
#include <type_traits>

#include "cp_f16_table.h"
#include "cp_launch.h"
#include "cp_resident.h"

namespace cp {

namespace {

typedef _Float16 h2 __attribute__((ext_vector_type(2)));

constexpr uint32_t kEnvsPerWave = 128u;
static_assert(kRowsBlockEnvs16 == 16u * kEnvsPerWave, "the rows blocks' 1,024 threads");

static_assert(f16tab::cosines_in_range(f16tab::make_table()),
              "a table cosine outside the range the reciprocals are keyed by");
// LDS layout: the divisor reciprocals, the reciprocals by cosine, then the
// sin/cos entries followed by entries of two NaNs (for NaN angles).
// The angle part spans every 14-bit pattern (|angle| bits & 0x3FFF), entries
// past 1/4 holding two NaNs: an angle within the limit indexes its own
// entry and a NaN angle (bits 0x7C01 .. 0x7FFF) one of the NaN entries.
// The two small tables come first, so that every table's byte offset fits
// the immediate offset of an LDS read.
constexpr uint32_t kAngleWords = 1u << 14;
constexpr uint32_t kDenWord = 0u;
constexpr uint32_t kRecipCosWord = kDenWord + f16tab::kDenEntries;
constexpr uint32_t kAngleWord = kRecipCosWord + f16tab::kCosEntries;
constexpr uint32_t kLutWords = (kAngleWord + kAngleWords + 3u) / 4u * 4u;

// The LDS image of the tables, evaluated at compile time.
struct Lut {
  alignas(16) uint32_t w[kLutWords];
};
constexpr Lut make_lut() {
  Lut l{};
  const f16tab::RecipTable den = f16tab::make_recip_table();
  const f16tab::RecipByCos cos = f16tab::make_recip_by_cos_table();
  const f16tab::Table angle = f16tab::make_table();
  for (uint32_t b = 0; b < kLutWords; ++b) l.w[b] = 0x7E007E00u;
  for (uint32_t b = 0; b < f16tab::kDenEntries; ++b) l.w[kDenWord + b] = __builtin_bit_cast(uint32_t, den.v[b]);
  for (uint32_t b = 0; b < f16tab::kCosEntries; ++b) l.w[kRecipCosWord + b] = __builtin_bit_cast(uint32_t, cos.v[b]);
  for (uint32_t b = 0; b < f16tab::kEntries; ++b) l.w[kAngleWord + b] = angle.v[b];
  return l;
}
__device__ const Lut kLut16 = make_lut();

__device__ __forceinline__ uint32_t bits(h2 v) { return __builtin_bit_cast(uint32_t, v); }
__device__ __forceinline__ h2 of_bits(uint32_t u) { return __builtin_bit_cast(h2, u); }

// RN16(a * c) for both halves of a (exact product, one rounding; the
// addend -0 keeps the sign of a zero product).
__device__ __forceinline__ h2 mul_round2(h2 a, float c) {
  uint32_t r;
  asm volatile("v_fma_mixlo_f16 %0, %1, %2, neg(0) op_sel_hi:[1,0,0]"
               : "=v"(r) : "v"(bits(a)), "v"(c));
  asm volatile("v_fma_mixhi_f16 %0, %1, %2, neg(0) op_sel:[1,0,0] op_sel_hi:[1,0,0]"
               : "+v"(r) : "v"(bits(a)), "v"(c));
  return of_bits(r);
}

// RN16(a[0] * c0) and RN16(a[1] * c1).
__device__ __forceinline__ h2 mul_round2(h2 a, float c0, float c1) {
  uint32_t r;
  asm volatile("v_fma_mixlo_f16 %0, %1, %2, neg(0) op_sel_hi:[1,0,0]"
               : "=v"(r) : "v"(bits(a)), "v"(c0));
  asm volatile("v_fma_mixhi_f16 %0, %1, %2, neg(0) op_sel:[1,0,0] op_sel_hi:[1,0,0]"
               : "+v"(r) : "v"(bits(a)), "v"(c1));
  return of_bits(r);
}

// RN16(a / m) for both halves, m the binary16 total mass, 1/m held as the sum
// of two binary16 numbers (Brisebarre, Muller and Raina 2004, as div_mass):
// the correctly rounded quotient for every finite binary16 |a| >= 0.0646
// (checked exhaustively).  Two packed operations where the mixed
// multiply-adds, a quarter-rate one for each half, cost as much as four.
constexpr double kInv16 = 1.0 / double(kTotalMass16);
constexpr half_t kInvHi16 = half_t(kInv16), kInvLo16 = half_t(kInv16 - double(kInvHi16));

__device__ __forceinline__ h2 div_mass2(h2 a) {
  return __builtin_elementwise_fma(a, h2{kInvHi16, kInvHi16}, a * h2{kInvLo16, kInvLo16});
}

typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));

// The LDS word at byte offset `off` of the table.
__device__ __forceinline__ uint32_t lut_at(const uint32_t *lut, uint32_t off) {
  return *reinterpret_cast<const uint32_t *>(reinterpret_cast<const char *>(lut) + off);
}

// RN32(1/d) for the divisors of the angular acceleration of both
// environments (the binary16 d in each half of db), from the LDS table: the
// index d - kDenFirst per half (16-bit arithmetic: wraps to large below
// kDenFirst), clamped to the last entry, which a NaN divisor reads (only
// with a NaN angle, whose numerator is NaN too).
__device__ __forceinline__ void recip2(uint32_t db, const uint32_t *lut, float &r0, float &r1) {
  u16x2 k = __builtin_bit_cast(u16x2, db) - u16x2{uint16_t(f16tab::kDenFirst), uint16_t(f16tab::kDenFirst)};
  k = __builtin_elementwise_min(k, u16x2{uint16_t(f16tab::kDenEntries - 1u), uint16_t(f16tab::kDenEntries - 1u)});
  const uint32_t off = __builtin_bit_cast(uint32_t, u16x2(k << uint16_t(2)));
  constexpr uint32_t kBase = 4u * kDenWord;
  r0 = __builtin_bit_cast(float, lut_at(lut, kBase + (off & 0xFFFFu)));
  r1 = __builtin_bit_cast(float, lut_at(lut, kBase + (off >> 16)));
}

// The same reciprocals from the cosines of both environments (cb: the
// binary16 cosines of the sin/cos table, each one of the 65 keys, or the NaN
// 0x7E00 of a NaN entry): byte offset (c - kCosFirst) * 4 mod 2^16, of which
// the low 9 bits are kept -- the keys' own offsets 0 .. 256, and for the NaN
// cosine 0x900 -> 0x100, the last key's entry, whose value does not matter
// there (that angle's numerator is NaN too).
__device__ __forceinline__ void recip2_by_cos(uint32_t cb, const uint32_t *lut, float &r0,
                                              float &r1) {
  constexpr uint16_t kFirst4 = uint16_t(f16tab::kCosFirst << 2);
  const uint32_t off = __builtin_bit_cast(
      uint32_t, u16x2(u16x2(__builtin_bit_cast(u16x2, cb) << uint16_t(2)) - u16x2{kFirst4, kFirst4}));
  constexpr uint32_t kBase = 4u * kRecipCosWord;
  r0 = __builtin_bit_cast(float, lut_at(lut, kBase + (off & 0x1FFu)));
  r1 = __builtin_bit_cast(float, lut_at(lut, kBase + ((off >> 16) & 0x1FFu)));
}

struct S2 {
  h2 x, xd, th, thd;
};

// sin and cos of both angles as the one-per-lane kernel computes them, for
// angles beyond the table (out of line: states the library produces never
// hold one after their first step).  Returns sin in the low and cos in the
// high half of each environment's word.
__device__ __attribute__((noinline)) uint64_t sincos2_beyond(uint32_t t) {
  half_t s0, c0, s1, c1;
  sincos16(__builtin_bit_cast(half_t, uint16_t(t)), s0, c0);
  sincos16(__builtin_bit_cast(half_t, uint16_t(t >> 16)), s1, c1);
  const uint32_t e0 = uint32_t(__builtin_bit_cast(uint16_t, s0)) |
                      (uint32_t(__builtin_bit_cast(uint16_t, c0)) << 16);
  const uint32_t e1 = uint32_t(__builtin_bit_cast(uint16_t, s1)) |
                      (uint32_t(__builtin_bit_cast(uint16_t, c1)) << 16);
  return (static_cast<uint64_t>(e1) << 32) | e0;
}

// sin and cos of both angles of th.  kAny: any angle (a launch's first
// step): from the table when every lane's angles are at most 1/4 in
// magnitude, else for the whole wave out of line.  Otherwise the angle is
// within the limit or NaN: the table alone, NaN reading an entry of NaNs.
template <bool kAny>
__device__ __forceinline__ void sincos2(h2 th, const uint32_t *lut, h2 &sn, h2 &c) {
  const uint32_t t = bits(th);
  const uint32_t a0 = t & 0x7FFFu, a1 = (t >> 16) & 0x7FFFu;
  uint32_t e0, e1;
  if (!kAny) {
    // both table offsets at once: the low 14 bits of each angle (an angle
    // within the limit is below 2^14, a NaN lands on a NaN entry), times 4
    const u16x2 a = __builtin_bit_cast(u16x2, t & 0x3FFF3FFFu);
    const uint32_t off = __builtin_bit_cast(uint32_t, u16x2(a << uint16_t(2)));
    e0 = lut_at(lut, 4u * kAngleWord + (off & 0xFFFFu));
    e1 = lut_at(lut, 4u * kAngleWord + (off >> 16));
    sn = of_bits(__builtin_amdgcn_perm(e1, e0, 0x05040100u) ^ (t & 0x80008000u));  // sin(-x) = -sin(x)
    c = of_bits(__builtin_amdgcn_perm(e1, e0, 0x07060302u));
    return;
  }
  if (__all(a0 <= f16tab::kLast && a1 <= f16tab::kLast)) {
    e0 = lut[kAngleWord + a0] ^ (t & 0x8000u);
    e1 = lut[kAngleWord + a1] ^ ((t >> 16) & 0x8000u);
  } else {
    const uint64_t e = sincos2_beyond(t);
    e0 = uint32_t(e);
    e1 = uint32_t(e >> 32);
  }
  sn = of_bits(__builtin_amdgcn_perm(e1, e0, 0x05040100u));
  c = of_bits(__builtin_amdgcn_perm(e1, e0, 0x07060302u));
}

// One explicit-Euler step of both environments, in the operation order of
// the binary16 step (dynamics16).  Past a launch's first step (kAny false) the
// old angle is within the limit, so an environment that goes on has |theta_dot|
// <= 0.419 / tau = 21: both dividends by m are then far from 0 (10 N less
// pml 21^2 sin 12 deg = 4.6, and pml |thacc| cos >= 0.2), where div_mass2 is
// exact.  One that ends its episode takes its start state, whatever its
// accelerations, which enter neither the new position nor the new angle.
template <bool kAny>
__device__ __forceinline__ S2 dynamics2(const S2 &s, h2 force, const uint32_t *lut) {
  const h2 g = h2{half_t(9.8), half_t(9.8)}, mp = h2{half_t(0.1), half_t(0.1)};
  const h2 l = h2{half_t(0.5), half_t(0.5)}, tau = h2{half_t(0.02), half_t(0.02)};
  const h2 four3 = h2{half_t(4.0 / 3.0), half_t(4.0 / 3.0)};
  const h2 pml = mp * l;
  h2 sn, c;
  sincos2<kAny>(s.th, lut, sn, c);
  const h2 thd2 = s.thd * s.thd;
  const h2 dividend = force + pml * thd2 * sn;
  const h2 temp = kAny ? mul_round2(dividend, kInvTotalMass16) : div_mass2(dividend);
  const h2 num = g * sn - c * temp;
  float r0, r1;
  if (kAny) {
    // any cosine: the divisor formed, its reciprocal looked up
    const h2 c2 = c * c;
    const h2 den = l * (four3 - mul_round2(mp * c2, kInvTotalMass16));
    recip2(bits(den), lut, r0, r1);
  } else {
    // a cosine from the table (or NaN): the reciprocal by the cosine
    recip2_by_cos(bits(c), lut, r0, r1);
  }
  const h2 thacc = mul_round2(num, r0, r1);
  const h2 part = pml * thacc * c;
  const h2 xacc = temp - (kAny ? mul_round2(part, kInvTotalMass16) : div_mass2(part));
  return S2{s.x + tau * s.xd, s.xd + tau * xacc, s.th + tau * s.thd, s.thd + tau * thacc};
}

// The lanes whose state is past a limit.
__device__ __forceinline__ unsigned long long done16(half_t x, half_t th) {
  const half_t xl = half_t(2.4), tl = half_t(kThetaLimit64);
  return __builtin_amdgcn_ballot_w64(__builtin_fabsf16(x) > xl) |
         __builtin_amdgcn_ballot_w64(__builtin_fabsf16(th) > tl);
}

// Prefetched start states of both environments, kept packed (x, x_dot,
// theta, theta_dot: one word each, environment 0 in the low half).
struct W4 {
  uint32_t x, xd, th, thd;
};

__device__ __forceinline__ uint32_t put16(uint32_t w, int h, half_t v) {
  const uint32_t b = __builtin_bit_cast(uint16_t, v);
  return h == 0 ? (w & 0xFFFF0000u) | b : (w & 0x0000FFFFu) | (b << 16);
}

// Start state of episode k of env into half `h` of n.
__device__ __forceinline__ void draw_into(W4 &n, int h, U2 key, uint32_t env, uint32_t k) {
  const State16 d = PrecF16::draw(key, env, k);
  n.x = put16(n.x, h, d.x);
  n.xd = put16(n.xd, h, d.xd);
  n.th = put16(n.th, h, d.th);
  n.thd = put16(n.thd, h, d.thd);
}

// The start state of episode k of env as two words of binary16 pairs:
// (x, x_dot) and (theta, theta_dot).
__device__ __forceinline__ void draw_words(U2 key, uint32_t env, uint32_t k, uint32_t &w0,
                                           uint32_t &w1) {
  const State16 d = PrecF16::draw(key, env, k);
  w0 = uint32_t(__builtin_bit_cast(uint16_t, d.x)) |
       (uint32_t(__builtin_bit_cast(uint16_t, d.xd)) << 16);
  w1 = uint32_t(__builtin_bit_cast(uint16_t, d.th)) |
       (uint32_t(__builtin_bit_cast(uint16_t, d.thd)) << 16);
}

// Half h of n from the words of draw_words.
__device__ __forceinline__ void put_words(W4 &n, int h, uint32_t w0, uint32_t w1) {
  if (h == 0) {
    n.x = __builtin_amdgcn_perm(n.x, w0, 0x07060100u);   // high half kept, low from w0.lo
    n.xd = __builtin_amdgcn_perm(n.xd, w0, 0x07060302u);  // low from w0.hi
    n.th = __builtin_amdgcn_perm(n.th, w1, 0x07060100u);
    n.thd = __builtin_amdgcn_perm(n.thd, w1, 0x07060302u);
  } else {
    n.x = __builtin_amdgcn_perm(w0, n.x, 0x05040100u);    // high from w0.lo, low kept
    n.xd = __builtin_amdgcn_perm(w0, n.xd, 0x07060100u);  // high from w0.hi
    n.th = __builtin_amdgcn_perm(w1, n.th, 0x05040100u);
    n.thd = __builtin_amdgcn_perm(w1, n.thd, 0x07060100u);
  }
}

// Keeps the compiler from moving memory accesses across this point (LDS
// exchanges within one wave, whose accesses the LDS executes in order).
__device__ __forceinline__ void lds_order() { asm volatile("" ::: "memory"); }

// Per-half select: the halves of r where m (0xFFFF per half) is set.
__device__ __forceinline__ h2 pick(uint32_t m, uint32_t r, h2 v) {
  return of_bits((r & m) | (bits(v) & ~m));
}

// kRows: as cp_resident.h, the block's pieces of the rows (3,000,001 x 50: 678
// us stored by waves, 554 by rows; aligned 449).
//
// A step is 50 issue slots (of a half-rate instruction) per 128 environments,
// the refills add 14; measured against the earlier form, with the actions read
// from the owning lanes, mixed multiply-adds for the divisions by m, and a test
// for a second termination at every step: 1,048,576 x 1,000 1,250 -> 993 us.
template <Traj kTraj, int kThreads>
__global__ __launch_bounds__(kThreads, kThreads == 1024 && kTraj != Traj::kRows ? 8 : 1) void k_resident_f16x2(RolloutParams p) {
  constexpr int kWaves = kThreads / 64;
  constexpr int kEnvs = kWaves * int(kEnvsPerWave);  // of a block
  __shared__ Lut tables;
  __shared__ uint32_t xch[kWaves][64][2];  // each wave's refill exchange
  __shared__ BlockTotals<kThreads> totals;
  __shared__ RowStage<half_t, kTraj == Traj::kRows ? kEnvs : 1> stages[2];
  totals.clear();
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
  for (uint32_t b = threadIdx.x; b < kLutWords / 4u; b += kThreads)
    reinterpret_cast<u32x4 *>(tables.w)[b] = reinterpret_cast<const u32x4 *>(kLut16.w)[b];
  const uint32_t *const lut = tables.w;
  __syncthreads();

  const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
  const uint32_t piece0 = (kTraj != Traj::kNone ? xcd_block() : blockIdx.x) * uint32_t(kEnvs);
  const uint32_t base = piece0 + wave * kEnvsPerWave;  // first env of the wave
  const uint32_t i0 = base + lane, i1 = base + 64u + lane;
  const bool v0 = i0 < p.n, v1 = i1 < p.n;
  half_t *const px = reinterpret_cast<half_t *>(p.x);
  half_t *const pxd = reinterpret_cast<half_t *>(p.xd);
  half_t *const pth = reinterpret_cast<half_t *>(p.th);
  half_t *const pthd = reinterpret_cast<half_t *>(p.thd);
  half_t *const pobs = reinterpret_cast<half_t *>(p.obs);
  const uint32_t e0 = p.env_base + i0, e1 = p.env_base + i1;
  uint32_t n_done_lane = 0u, returns = 0u;
  // Waves wholly past the batch skip the loop (they still take part in the
  // block's totals), where the block's waves do not wait for each other.
  if (base < p.n || kTraj != Traj::kNone) {
    // environments past the batch: at rest for the first step, whose angles
    // beyond the table are evaluated out of line, then NaN states, which never
    // end an episode (cp_resident.h)
    const half_t rest = half_t(0.0), nan = half_t(__builtin_nanf(""));
    S2 s{h2{rest, rest}, h2{rest, rest}, h2{rest, rest}, h2{rest, rest}};
    uint32_t k[2] = {0u, 0u};
    if (v0) {
      s.x[0] = px[i0]; s.xd[0] = pxd[i0]; s.th[0] = pth[i0]; s.thd[0] = pthd[i0];
      k[0] = p.ep_index[i0];
    }
    if (v1) {
      s.x[1] = px[i1]; s.xd[1] = pxd[i1]; s.th[1] = pth[i1]; s.thd[1] = pthd[i1];
      k[1] = p.ep_index[i1];
    }
    // Episode counters are brought up to date at the refills only: an
    // environment whose bit of used0 / used1 is set ended an episode since the
    // last refill and is in episode k + 1 (cp_resident.h).  last: the step (of
    // this launch, below 2^16) of the latest termination of each environment,
    // in the halves of one word.
    uint32_t last = 0u;
    unsigned long long used0 = 0u, used1 = 0u;
    W4 nxt{0u, 0u, 0u, 0u};  // next start states, drawn ahead of time
    draw_into(nxt, 0, p.krst, e0, k[0] + 1u);
    draw_into(nxt, 1, p.krst, e1, k[1] + 1u);
    // Random actions (cp_resident.h, HashPolicy): both environments' actions
    // of 16 steps in the halves of one word, the next step's in the halves'
    // top bits; the words of 64 steps in turn.
    const uint32_t g0 = uint32_t(__builtin_amdgcn_readfirstlane(int(e0))) >> 6;
    uint32_t act[4];
    auto prepare = [&](uint32_t t, bool first) {
      if (first || (t & 63u) == 0u) {
        const uint32_t step = (t & ~63u) + (lane ^ 31u);
        U2 b0 = threefry2x32(p.kact.a, p.kact.b, g0, step);
        U2 b1 = threefry2x32(p.kact.a, p.kact.b, g0 + 1u, step);
        transpose64(b0.a, b0.b);
        transpose64(b1.a, b1.b);
        act[0] = __builtin_amdgcn_perm(b1.a, b0.a, 0x07060302u);
        act[1] = __builtin_amdgcn_perm(b1.a, b0.a, 0x05040100u);
        act[2] = __builtin_amdgcn_perm(b1.b, b0.b, 0x07060302u);
        act[3] = __builtin_amdgcn_perm(b1.b, b0.b, 0x05040100u);
        for (uint32_t q = (t >> 4) & 3u; q > 0u; --q) {  // only at a launch's first step
          act[0] = act[1]; act[1] = act[2]; act[2] = act[3];
        }
        act[0] <<= t & 15u;
      } else if ((t & 15u) == 0u) {
        act[0] = act[1]; act[1] = act[2]; act[2] = act[3];
      }
    };
    half_t *row_obs = pobs;
    float *row_reward = p.reward;
    uint8_t *row_done = p.done;
    uint32_t turn = 0u;
    const bool whole = piece0 + uint32_t(kEnvs) <= p.n;
    uint32_t jj = 0u;  // the step (of this launch) in both halves
    auto step = [&](auto any) {
      const h2 force = of_bits((act[0] & 0x80008000u) ^ 0xC900C900u);  // -10, or 10 where the bit is set
      act[0] <<= 1;  // the low half's bits reach the high half's top after its 16 are used
      S2 o = dynamics2<decltype(any)::value>(s, force, lut);
      const unsigned long long m0 = done16(o.x[0], o.th[0]), m1 = done16(o.x[1], o.th[1]);
      const bool d0 = __builtin_amdgcn_inverse_ballot_w64(m0), d1 = __builtin_amdgcn_inverse_ballot_w64(m1);
      const uint32_t m = (d0 ? 0x0000FFFFu : 0u) | (d1 ? 0xFFFF0000u : 0u);
      last = (last & ~m) | (jj & m);
      jj += 0x00010001u;
      o.x = pick(m, nxt.x, o.x);
      o.xd = pick(m, nxt.xd, o.xd);
      o.th = pick(m, nxt.th, o.th);
      o.thd = pick(m, nxt.thd, o.thd);
      used0 |= m0;
      used1 |= m1;
      s = o;
      if constexpr (kTraj == Traj::kRows) {
        RowStage<half_t, kEnvs> &st = stages[turn];
        turn ^= 1u;
        const h2 v[4] = {s.x, s.xd, s.th, s.thd};
        const uint32_t q0 = wave * kEnvsPerWave + lane, q1 = q0 + 64u;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          st.v[c][q0] = v[c][0];
          st.v[c][q1] = v[c][1];
        }
        st.done[q0] = uint8_t(d0);
        st.done[q1] = uint8_t(d1);
        __syncthreads();
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const uint32_t at = uint32_t(h * kThreads);
#pragma unroll
          for (uint32_t c = 0; c < 4u; ++c) {
            half_t *const piece = row_obs + size_t(c) * p.n + piece0;
            const uint32_t e = turned<kEnvs>(piece, 2u, at);
            if (whole || piece0 + e < p.n) *elem<true>(piece, e) = st.v[c][e];
          }
          float *const piece_r = row_reward + piece0;
          const uint32_t er = turned<kEnvs>(piece_r, 4u, at);
          if (whole || piece0 + er < p.n) *elem<true>(piece_r, er) = 1.0f;
          uint8_t *const piece_d = row_done + piece0;
          const uint32_t ed = turned<kEnvs>(piece_d, 1u, at);
          if (whole || piece0 + ed < p.n) *elem<true>(piece_d, ed) = st.done[ed];
        }
      } else if constexpr (kTraj != Traj::kNone) {
        constexpr bool kAll = kTraj == Traj::kAll;  // (32-bit offsets then)
        if (v0) store_traj<kAll, kAll>(row_obs, row_reward, row_done, p.n, i0,
                                       State16{s.x[0], s.xd[0], s.th[0], s.thd[0]}, d0);
        if (v1) store_traj<kAll, kAll>(row_obs, row_reward, row_done, p.n, i1,
                                       State16{s.x[1], s.xd[1], s.th[1], s.thd[1]}, d1);
      }
      if constexpr (kTraj != Traj::kNone) {
        if (kTraj >= Traj::kAll || row_obs) row_obs += 4u * size_t(p.n);
        if (kTraj >= Traj::kAll || row_reward) row_reward += p.n;
        if (kTraj >= Traj::kAll || row_done) row_done += p.n;
      }
    };
    // The refill after a round: the environments that used their prefetched
    // start state (about a third of them after 8 steps) get the next one.
    // Their requests (environment, episode) are packed into consecutive
    // slots of the wave's exchange area in LDS, lane r of the wave draws
    // request r -- one generator pass for up to 64 requests, instead of one
    // pass for each half whenever any of its lanes asks -- and the
    // requesting lanes read their start states back.  The slots of a wave are
    // its own and the LDS executes a wave's accesses in program order, so
    // only the compiler's ordering needs fixing (lds_order).
    auto refill = [&]() {
      const unsigned long long m0 = used0, m1 = used1;
      if ((m0 | m1) == 0u) return;
      used0 = used1 = 0u;
      const bool mine0 = __builtin_amdgcn_inverse_ballot_w64(m0), mine1 = __builtin_amdgcn_inverse_ballot_w64(m1);
      const uint32_t c0 = uint32_t(__popcll(m0)), total = c0 + uint32_t(__popcll(m1));
      const uint32_t s0 = __builtin_amdgcn_mbcnt_hi(uint32_t(m0 >> 32), __builtin_amdgcn_mbcnt_lo(uint32_t(m0), 0u));
      const uint32_t s1 = c0 + __builtin_amdgcn_mbcnt_hi(uint32_t(m1 >> 32), __builtin_amdgcn_mbcnt_lo(uint32_t(m1), 0u));
      if (mine0) k[0] += 1u;
      if (mine1) k[1] += 1u;
      uint32_t(*const slot)[2] = xch[wave];
      for (uint32_t base = 0; base < total; base += 64u) {
        if (mine0 && s0 - base < 64u) {
          slot[s0 - base][0] = e0;
          slot[s0 - base][1] = k[0] + 1u;
        }
        if (mine1 && s1 - base < 64u) {
          slot[s1 - base][0] = e1;
          slot[s1 - base][1] = k[1] + 1u;
        }
        lds_order();
        uint32_t w0 = 0u, w1 = 0u;
        if (base + lane < total) draw_words(p.krst, slot[lane][0], slot[lane][1], w0, w1);
        lds_order();
        slot[lane][0] = w0;
        slot[lane][1] = w1;
        lds_order();
        if (mine0 && s0 - base < 64u) put_words(nxt, 0, slot[s0 - base][0], slot[s0 - base][1]);
        if (mine1 && s1 - base < 64u) put_words(nxt, 1, slot[s1 - base][0], slot[s1 - base][1]);
        lds_order();
      }
    };
    using any_angle = std::integral_constant<bool, true>;
    using limited_angle = std::integral_constant<bool, false>;
    // groups of steps as in the one-per-lane loop (cp_resident.h), each but the
    // last followed by a refill
    uint32_t j = 1u;
    prepare(p.t0, true);
    step(any_angle{});
    if (!v0) s.x[0] = s.xd[0] = s.th[0] = s.thd[0] = nan;
    if (!v1) s.x[1] = s.xd[1] = s.th[1] = s.thd[1] = nan;
    const uint32_t lead = (0u - (p.t0 + 1u)) & (kRefill - 1u);
    for (const uint32_t end = p.T < 1u + lead ? p.T : 1u + lead; j < end; ++j) step(limited_angle{});
    if (j < p.T) refill();
    // A trajectory's waves go on together, neighbours on one XCD, so that the
    // parts of lines that they store meet in its L2: after every eight steps
    // (3,000,000 x 50 491 -> 449 us, 4,194,304 x 50 684 -> 608, 1,000,000 x 50
    // 169 -> 148), the large blocks also after the first group and every four
    // (2,000,003 x 17 164 -> 152, 1,000,003 x 76 302 -> 288, 4,000,000 x 8 152
    // -> 132; in the small ones it would cost 20,001 x 769 343 -> 365).
    auto together = [&](bool round) {
      if ((kTraj == Traj::kAny || kTraj == Traj::kAll) && (round || kThreads == 1024)) __syncthreads();
    };
    together(false);
    while (j + kRefill <= p.T) {
      prepare(p.t0 + j, false);
#pragma unroll(kTraj == Traj::kNone ? 4 : 1)
      for (uint32_t r = 0; r < kRefill; ++r) {
        step(limited_angle{});
        if (r == kRefill / 2u - 1u) together(false);
      }
      j += kRefill;
      if (j < p.T) refill();
      together(true);
    }
    if (j < p.T) {
      prepare(p.t0 + j, false);
      for (; j < p.T; ++j) step(limited_angle{});
    }
    if (__builtin_amdgcn_inverse_ballot_w64(used0)) k[0] += 1u;
    if (__builtin_amdgcn_inverse_ballot_w64(used1)) k[1] += 1u;
    // as the one-per-lane kernel: the episode length at the end is the steps
    // since the latest termination, or the starting length plus T without one,
    // terminations are the growth of the episode index, finished returns
    // T + len(start) - len(end); the starting counters are still in memory
    const bool v[2] = {v0, v1};
    const uint32_t ii[2] = {i0, i1};
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      if (!v[h]) continue;
      const uint32_t i = ii[h];
      const uint32_t k0 = p.ep_index[i], len0 = p.ep_len[i];
      const uint32_t l = h == 0 ? last & 0xFFFFu : last >> 16;
      const uint32_t len = k[h] != k0 ? p.T - 1u - l : len0 + p.T;
      const uint32_t n_done = k[h] - k0, ret = p.T + len0 - len;
      n_done_lane += n_done;
      returns += ret;
      px[i] = s.x[h];
      pxd[i] = s.xd[h];
      pth[i] = s.th[h];
      pthd[i] = s.thd[h];
      p.ep_index[i] = k[h];
      p.ep_len[i] = len;
      if (p.done_count) p.done_count[i] = (p.first ? 0u : p.done_count[i]) + n_done;
      if (p.total_reward) {
        const float prev = p.first ? 0.0f : p.total_reward[i];
        const float cap = float(1u << 24);
        p.total_reward[i] = prev >= cap ? prev : __builtin_fminf(prev + float(p.T), cap);
      }
      if (p.ret_sum) p.ret_sum[i] = (p.first ? 0u : p.ret_sum[i]) + ret;
    }
  }
  if (p.global) totals.publish(p.global, n_done_lane, returns);
}

}  // namespace

bool resident_f16x2_applies(const RolloutParams &p) { return p.env_base % 64u == 0u; }

// Blocks of 1,024 threads (2,048 environments), two per CU, share a copy of
// the tables among 16 waves.  Batches that blocks of 256 spread over the CUs
// once, at two per CU, take those: 200 steps of 1,024 environments 91.5 -> 48.1
// us, of 100,003 144 -> 52, of 262,144 146 -> 72 (of 300,000, in blocks of
// 1,024, 146 -> 119, for the shorter step).
constexpr uint32_t kSmallBlocksMaxEnvs = 262144;

template <Traj kTraj, int kThreads>
static void f16x2_as(const RolloutParams &p, hipStream_t stream) {
  const uint32_t per_block = uint32_t(kThreads) * 2u;
  hipLaunchKernelGGL((k_resident_f16x2<kTraj, kThreads>), dim3((p.n + per_block - 1u) / per_block),
                     dim3(kThreads), 0, stream, p);
}

// At most 2^16 steps per launch (the kernel keeps step indices in 16-bit
// halves); a longer rollout is split into launches the way steps_per_launch
// splits one, which changes no result.
constexpr uint32_t kMaxStepsF16x2 = 1u << 16;

template <Traj kTraj>
static void f16x2_sized(const RolloutParams &p, hipStream_t stream) {
  if (p.n <= kSmallBlocksMaxEnvs) f16x2_as<kTraj, 256>(p, stream);
  else f16x2_as<kTraj, 1024>(p, stream);
}

hipError_t launch_resident_f16x2(const RolloutParams &p, hipStream_t stream) {
  for (uint64_t j = 0; j < p.T; j += kMaxStepsF16x2) {
    RolloutParams q = p;
    q.t0 = p.t0 + uint32_t(j);
    q.T = uint32_t(p.T - j < kMaxStepsF16x2 ? p.T - j : kMaxStepsF16x2);
    q.first = p.first && j == 0u;
    // trajectory rows: 4 * n binary16 obs values, n rewards, n flags per step
    if (p.obs) q.obs = reinterpret_cast<float *>(reinterpret_cast<half_t *>(p.obs) + size_t(j) * 4u * p.n);
    if (p.reward) q.reward = p.reward + size_t(j) * p.n;
    if (p.done) q.done = p.done + size_t(j) * p.n;
    if (rows_block(q, sizeof(half_t)) != 0u) {
      f16x2_as<Traj::kRows, 1024>(q, stream);
    } else {
      switch (traj_kind(q, sizeof(half_t))) {
        case Traj::kNone: f16x2_sized<Traj::kNone>(q, stream); break;
        case Traj::kAny: f16x2_sized<Traj::kAny>(q, stream); break;
        default: f16x2_sized<Traj::kAll>(q, stream); break;
      }
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace cp

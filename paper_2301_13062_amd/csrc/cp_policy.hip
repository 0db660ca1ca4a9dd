// cp_policy.hip -- register-resident rollout whose actions come from a
// 4-64-64-2 tanh MLP policy evaluated on the matrix cores, the simulation
// and the network inference fused in one kernel (the paper's first
// future-work item, Sec. "Future Work").
//
// A wave holds 16, 32 or 64 environments as one, two or four tiles of 16
// (with fewer than four tiles the lane groups past them repeat the first
// ones' environments), and evaluates the policy tile by tile, two at a time
// where it has them (two independent chains of matrix products and tanh for
// the scheduler to interleave).  Every dense layer is a chain of
// v_mfma_f32_16x16x16_bf16 with the weights as the A operand (neurons =
// rows) and the environments as the B operand (columns): lane 16g+c holds
// A[c][4g..4g+3], B[4g..4g+3][c] and D[4g..4g+3][c].  Since a layer's D
// layout (4 consecutive neurons of environment c per lane) is exactly the
// next layer's B layout (4 consecutive K indices of column c), the hidden
// activations go from accumulator to tanh to bf16 to the next MFMA without
// leaving the lane.  Nothing crosses lanes but the chosen actions' lane
// masks: lane 16g+c owns environment c of tile g and passes its observation
// as K indices 4g..4g+3 of that tile's layer 1 (W1 repeated for every g, the
// other lane groups' B values zero), and the rows of W3 are repeated for every
// g, so that every group receives the logits.  The 8,960 bytes of bf16
// weights are staged once per block in LDS; the layer-1 and layer-3
// fragments are then held in registers, the 16 layer-2 fragments are read
// from LDS at every use (held in registers they would leave room for one
// tile at a time only).
#include "cp_launch.h"
#include "cp_resident.h"

namespace cp {

namespace {

typedef short bf16x4 __attribute__((ext_vector_type(4)));  // four bf16 bit patterns
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kIn = 4, kHid = 64, kOut = 2;
constexpr int kOffW1 = 0, kOffW2 = kIn * kHid, kOffW3 = kOffW2 + kHid * kHid;
constexpr int kWeights = kOffW3 + kHid * kOut;  // 4480
static_assert(kWeights == 4480, "weight count");

// tanh in binary32 for an activation that is rounded to bfloat16 next:
// x P(x^2) / Q(x^2) with P and Q of degree 3 (a rational fit on [0, 3.5] by
// iteratively reweighted linearised least squares, of relative error 1.9e-9,
// 6.5e-9 with its coefficients in binary32), evaluated with one hardware
// reciprocal: within about 0.7 ulp
// on average and 4.3 at most.  From atanh(1 - 2^-9) = 3.466 on, tanh rounds
// to bfloat16 +-1 (its bfloat16 neighbour below 1 is 1 - 2^-8), and so does
// the fit from there to 9.64 (0.99806 .. 1.0039): an argument known to be at
// most kTanhFree needs no clamp (kClamp false), any other is clamped to
// +-3.5, with the same rounded activation.  Over 24 million arguments its
// bfloat16 roundings differ from those of the exact tanh no more often (1 in
// 10^5) than a degree-4 fit on [0, 9] did, with two fewer multiply-adds per
// evaluation.
constexpr float kTanhFree = 9.5f;

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

typedef float f32x2 __attribute__((ext_vector_type(2)));

// Two binary32 values -> two bfloat16 (round to nearest, ties to even) in
// one dword, low half first: one v_cvt_pk_bf16_f32.
__device__ __forceinline__ uint32_t pack2(float lo, float hi) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{lo, hi}, bf16x2));
}

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// Two dwords of packed bfloat16 pairs as one MFMA operand (no data movement).
__device__ __forceinline__ bf16x4 as_bf16x4(uint32_t lo, uint32_t hi) {
  return __builtin_bit_cast(bf16x4, u32x2{lo, hi});
}

// out = bf16(tanh(acc)) for kN accumulators, stage by stage over their 4 kN
// values, which keeps as many independent chains in flight (a wave alone on
// its SIMD waits out every dependence: 64 steps of 10,007 environments, one
// tile per wave, 80 -> 75 us; 4,194,304 x 64: 10.35 -> 9.66 ms).
template <bool kClamp, int kN>
__device__ __forceinline__ void tanh_bf16(const f32x4 (&acc)[kN], bf16x4 (&out)[kN]) {
  constexpr int kV = 4 * kN;
  float x[kV], z[kV], p[kV], q[kV];
#pragma unroll
  for (int v = 0; v < kV; ++v)
    x[v] = kClamp ? __builtin_amdgcn_fmed3f(acc[v / 4][v % 4], -3.5f, 3.5f) : acc[v / 4][v % 4];
#pragma unroll
  for (int v = 0; v < kV; ++v) z[v] = x[v] * x[v];
#pragma unroll
  for (int v = 0; v < kV; ++v) q[v] = __builtin_fmaf(0x1.8752cep-13f, z[v], 0x1.73e8d6p-6f);
#pragma unroll
  for (int v = 0; v < kV; ++v) q[v] = __builtin_fmaf(q[v], z[v], 0x1.d7335ep-2f);
#pragma unroll
  for (int v = 0; v < kV; ++v) q[v] = __builtin_fmaf(q[v], z[v], 1.0f);
#pragma unroll
  for (int v = 0; v < kV; ++v) p[v] = __builtin_fmaf(0x1.9b61d8p-18f, z[v], 0x1.5af996p-9f);
#pragma unroll
  for (int v = 0; v < kV; ++v) q[v] = __builtin_amdgcn_rcpf(q[v]);
#pragma unroll
  for (int v = 0; v < kV; ++v) p[v] = __builtin_fmaf(p[v], z[v], 0x1.03bc14p-3f);
#pragma unroll
  for (int v = 0; v < kV; ++v) p[v] = __builtin_fmaf(p[v], z[v], 1.0f);
#pragma unroll
  for (int v = 0; v < kV; ++v) p[v] = (x[v] * p[v]) * q[v];
#pragma unroll
  for (int v = 0; v < kN; ++v)
    out[v] = as_bf16x4(pack2(p[4 * v], p[4 * v + 1]), pack2(p[4 * v + 2], p[4 * v + 3]));
}

__device__ __forceinline__ f32x4 mma(bf16x4 a, bf16x4 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, 0, 0, 0);
}

// Layer-2 weight fragments in LDS in the order the lanes read them:
// fragment (m, kc) of lane L (rows 16m.., K chunk 16kc.. of W2^T) at
// [(4m + kc) * 64 + L], 8 bytes, so that a wave reads one fragment with one
// conflict-free ds_read_b64.  `w` is the staged row-major [in][out] array.
constexpr int kW2Frags = 16 * 64;

__device__ __forceinline__ void stage_w2_fragments(const uint16_t *w, bf16x4 *w2f) {
  for (int idx = threadIdx.x; idx < kW2Frags; idx += kResidentBlock) {
    const int mk = idx >> 6, lane = idx & 63, m = mk >> 2, kc = mk & 3;
    const int g = lane >> 4, c = lane & 15;
    bf16x4 f;
    for (int j = 0; j < 4; ++j) f[j] = short(w[kOffW2 + (16 * kc + 4 * g + j) * kHid + 16 * m + c]);
    w2f[idx] = f;
  }
}

// The staged weights of a block and the sizes of its layers' sums.
struct MlpStage {
  alignas(16) uint16_t w[kWeights];
  bf16x4 w2f[kW2Frags];
  float col[kResidentWaves][kHid];  // sums of |W2[k][m]| over each wave's k
};

__device__ __forceinline__ float bf16_value(uint16_t u) {
  return __builtin_bit_cast(float, uint32_t(u) << 16);
}

// Every thread of the block: stages the weights and returns the largest sum
// |x| + |x_dot| + |theta| + |theta_dot| of an environment for which no
// argument of a tanh can pass kTanhFree -- layer 1: that sum times the
// largest |W1|, with 1% for the rounding of the inputs; layer 2, whose inputs
// are at most 1 in magnitude: the largest column sum of |W2| -- or -1 if
// layer 2's may (or a weight is not finite).
__device__ __forceinline__ float stage_weights(const uint16_t *__restrict__ policy_w, MlpStage &st) {
  if ((reinterpret_cast<uintptr_t>(policy_w) & 15u) == 0u) {
    // 560 16-byte pieces, three loads in flight per lane
    const u32x4 *src = reinterpret_cast<const u32x4 *>(policy_w);
    u32x4 *dst = reinterpret_cast<u32x4 *>(st.w);
    constexpr int kPieces = kWeights / 8, kRounds = (kPieces + kResidentBlock - 1) / kResidentBlock;
    u32x4 v[kRounds];
#pragma unroll
    for (int r = 0; r < kRounds; ++r)
      if (r * kResidentBlock + int(threadIdx.x) < kPieces) v[r] = src[r * kResidentBlock + threadIdx.x];
#pragma unroll
    for (int r = 0; r < kRounds; ++r)
      if (r * kResidentBlock + int(threadIdx.x) < kPieces) dst[r * kResidentBlock + threadIdx.x] = v[r];
  } else {
    for (int idx = threadIdx.x; idx < kWeights; idx += kResidentBlock) st.w[idx] = policy_w[idx];
  }
  __syncthreads();
  stage_w2_fragments(st.w, st.w2f);
  // wave v sums rows 16v .. 16v + 15 of column `lane`
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  constexpr int kRows = kHid / kResidentWaves;
  float sum = 0.0f;
#pragma unroll
  for (int k = 0; k < kRows; ++k)
    sum += __builtin_fabsf(bf16_value(st.w[kOffW2 + (kRows * wave + k) * kHid + lane]));
  st.col[wave][lane] = sum;
  float w1 = 0.0f;
#pragma unroll
  for (int k = 0; k < kIn; ++k) w1 = fmaxf(w1, __builtin_fabsf(bf16_value(st.w[kOffW1 + k * kHid + lane])));
  __syncthreads();
  float w2 = 0.0f;
#pragma unroll
  for (int v = 0; v < kResidentWaves; ++v) w2 += st.col[v][lane];
  // (a NaN fails this comparison; fmaxf would drop it)
  const bool bounded = __all(w2 <= kTanhFree);
  // likewise for W1: a NaN or infinite weight makes the sum below not finite
  float all = 0.0f;
#pragma unroll
  for (int k = 0; k < kIn; ++k) all += bf16_value(st.w[kOffW1 + k * kHid + lane]) * 0.0f;
#pragma unroll
  for (int k = 0; k < kOut; ++k) all += bf16_value(st.w[kOffW3 + lane * kOut + k]) * 0.0f;
  const bool finite = __all(all == 0.0f);
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) w1 = fmaxf(w1, __shfl_xor(w1, off, 64));
  return bounded && finite ? kTanhFree / (1.01f * w1 + 1e-30f) : -1.0f;
}

// kTiles: tiles of 16 environments per wave (1, 2 or 4).
template <int kTiles>
struct MlpPolicy {
  // one copy of a step's code in the loop: eight would not fit the
  // instruction cache
  static constexpr bool kUnrolled = false;
  static constexpr bool kBlockRefill = false;  // bound by the network, not by stores
  static constexpr bool kAhead = false;
  static constexpr uint32_t kEnvsPerWave = 16u * kTiles;
  static constexpr int kPair = kTiles > 1 ? 2 : 1;  // tiles in flight
  // One tile per wave (at most three waves per SIMD): all of layer 2's row
  // blocks in flight and its weights in registers.
  static constexpr bool kHoldW2 = kTiles == 1;
  static constexpr int kRows = kTiles == 1 ? 4 : 1;

  bf16x4 w1[4];       // W1^T rows 16m..16m+15, K = the 4 inputs (for every lane group)
  bf16x4 w3[4];       // W3^T rows 0,1 repeated as 4g, 4g+1 (lanes c % 4 < 2), K chunk 16c..
  const bf16x4 *w2f;  // W2^T fragments in LDS (stage_w2_fragments)
  bf16x4 w2[kHoldW2 ? 16 : 1];  // ... held
  float free_sum;     // stage_weights
  bool past;          // a lane past the batch: its (NaN) state decides nothing

  // Fragments from the staged weights (row-major [in][out] bf16).
  __device__ __forceinline__ void load(const MlpStage &st, float free, bool past_batch) {
    const uint32_t lane = threadIdx.x & 63u, g = lane >> 4, c = lane & 15u;
    w2f = st.w2f;
    if (kHoldW2)
      for (int f = 0; f < (kHoldW2 ? 16 : 1); ++f) w2[f] = w2f[f * 64 + lane];
    free_sum = free;
    past = past_batch;
    for (int m = 0; m < 4; ++m) {
      for (int j = 0; j < 4; ++j) w1[m][j] = short(st.w[kOffW1 + j * kHid + 16 * m + c]);
      for (int j = 0; j < 4; ++j)
        w3[m][j] = (c & 3u) < 2u ? short(st.w[kOffW3 + (16 * m + 4 * g + j) * kOut + (c & 3u)]) : short(0);
    }
  }

  template <Group>
  __device__ __forceinline__ void prepare(uint32_t) {}

  // The hidden activations of row blocks mp .. mp + kRows - 1.
  template <bool kClamp>
  __device__ __forceinline__ static void activate(const f32x4 (&acc)[kRows * kPair],
                                                  bf16x4 (&h)[4][kPair], int mp) {
    bf16x4 out[kRows * kPair];
    tanh_bf16<kClamp>(acc, out);
#pragma unroll
    for (int m = 0; m < kRows; ++m)
#pragma unroll
      for (int q = 0; q < kPair; ++q) h[mp + m][q] = out[m * kPair + q];
  }

  // The lanes whose environment is pushed right, for its pre-step state s.
  // kClamp false: no tanh argument passes kTanhFree, every value is finite.
  template <bool kClamp>
  __device__ __forceinline__ unsigned long long evaluate(const State &s) const {
    const uint32_t lane = threadIdx.x & 63u, g = lane >> 4, c = lane & 15u;
    const uint32_t o01 = pack2(s.x, s.xd), o23 = pack2(s.th, s.thd);
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    const bf16x4 none = as_bf16x4(0u, 0u);
    unsigned long long right = 0u;
#pragma unroll
    for (int tp = 0; tp < kTiles; tp += kPair) {
      bf16x4 in[kPair];
#pragma unroll
      for (int q = 0; q < kPair; ++q) {
        if (kClamp) {
          // from the lane that owns the environment to lane group 0, so that
          // no product of a zero and an infinite weight enters the sum
          const int src = int(16 * (tp + q) + c) * 4;
          const uint32_t b01 = uint32_t(__builtin_amdgcn_ds_bpermute(src, int(o01)));
          const uint32_t b23 = uint32_t(__builtin_amdgcn_ds_bpermute(src, int(o23)));
          in[q] = g == 0u ? as_bf16x4(b01, b23) : none;
        } else {
          in[q] = g == uint32_t(tp + q) ? as_bf16x4(o01, o23) : none;
        }
      }
      bf16x4 h1[4][kPair], h2[4][kPair];
#pragma unroll
      for (int mp = 0; mp < 4; mp += kRows) {
        f32x4 acc[kRows * kPair];
#pragma unroll
        for (int m = 0; m < kRows; ++m) {
          const bf16x4 wf = kClamp && g != 0u ? none : w1[mp + m];
#pragma unroll
          for (int q = 0; q < kPair; ++q) acc[m * kPair + q] = mma(wf, in[q], zero);
        }
        activate<kClamp>(acc, h1, mp);
      }
#pragma unroll
      for (int mp = 0; mp < 4; mp += kRows) {
        f32x4 acc[kRows * kPair];
#pragma unroll
        for (int v = 0; v < kRows * kPair; ++v) acc[v] = zero;
        // an opaque offset keeps the compiler from hoisting the fragment
        // reads out of the step loop into registers
        uint32_t off = lane;
        if (!kHoldW2) asm volatile("" : "+v"(off));
#pragma unroll
        for (int kc = 0; kc < 4; ++kc)
#pragma unroll
          for (int m = 0; m < kRows; ++m) {
            const int f = 4 * (mp + m) + kc;
            const bf16x4 wf = kHoldW2 ? w2[kHoldW2 ? f : 0] : w2f[f * 64 + off];
#pragma unroll
            for (int q = 0; q < kPair; ++q)
              acc[m * kPair + q] = mma(wf, h1[kc][q], acc[m * kPair + q]);
          }
        activate<kClamp>(acc, h2, mp);
      }
#pragma unroll
      for (int q = 0; q < kPair; ++q) {
        f32x4 logits = zero;
#pragma unroll
        for (int kc = 0; kc < 4; ++kc) logits = mma(w3[kc], h2[kc][q], logits);
        // every group's rows 4g and 4g + 1: the logits of environment c of
        // this tile, whose lanes take them
        constexpr unsigned long long kLanes = kTiles == 1   ? ~0ull
                                              : kTiles == 2 ? 0x0000FFFF0000FFFFull
                                                            : 0xFFFFull;
        right |= __builtin_amdgcn_ballot_w64(logits[1] > logits[0]) & (kLanes << (16 * (tp + q)));
      }
    }
    return right;
  }

  // Action of the lane's environment for its pre-step state s, in the top bit.  Called by
  // every lane of the wave.  The clamp is a half-rate instruction, a seventh
  // of a tanh's issue time; every wave of the usual networks and states goes
  // without (4,194,304 x 64: 11.06 -> 10.32 ms).
  __device__ __forceinline__ uint32_t operator()(const State &s) const {
    const float sum = (__builtin_fabsf(s.x) + __builtin_fabsf(s.xd)) +
                      (__builtin_fabsf(s.th) + __builtin_fabsf(s.thd));
    const unsigned long long right = __all(sum <= free_sum || past) ? evaluate<false>(s) : evaluate<true>(s);
    return __builtin_amdgcn_inverse_ballot_w64(right) ? 0x80000000u : 0u;
  }
};

template <Traj kTraj, int kTiles>
__global__ __launch_bounds__(kResidentBlock, kTiles == 1 ? 2 : 1) void k_resident_policy(RolloutParams p) {
  __shared__ MlpStage stage;
  const float free = stage_weights(p.policy_w, stage);
  MlpPolicy<kTiles> policy;
  policy.load(stage, free, lane_env<MlpPolicy<kTiles>>(blockIdx.x) >= p.n);
  resident_rollout<kTraj>(p, policy, blockIdx.x);
}

// The policy alone (simulation and inference as separate kernels, the
// alternative to fusing them): actions[i] = the MLP's action for the state
// obs[0..3][i].  Blocks stage the weights once and stride over the batch;
// lanes past the batch evaluate the last environment (every lane of a wave
// takes part in the cross-lane exchanges) and store nothing.
template <int kTiles>
__global__ __launch_bounds__(kResidentBlock, kTiles == 1 ? 2 : 1) void k_policy_actions(
    const float *__restrict__ obs, uint32_t n, const uint16_t *__restrict__ policy_w,
    uint8_t *__restrict__ actions) {
  using Policy = MlpPolicy<kTiles>;
  constexpr uint32_t kEnvs = kResidentWaves * Policy::kEnvsPerWave;  // per block and round
  __shared__ MlpStage stage;
  const float free = stage_weights(policy_w, stage);
  Policy policy;
  policy.load(stage, free, false);
  const bool owner = (threadIdx.x & 63u) < Policy::kEnvsPerWave;
  for (uint32_t i = lane_env<Policy>(blockIdx.x), base = blockIdx.x * kEnvs; base < n;
       base += gridDim.x * kEnvs, i += gridDim.x * kEnvs) {
    const uint32_t ic = i < n ? i : n - 1u;
    // plane offsets in 64 bits: 3n passes 2^32 from n > 1,431,655,765
    const size_t m = n;
    const State s{obs[ic], obs[m + ic], obs[2u * m + ic], obs[3u * m + ic]};
    const uint32_t a = policy(s);
    if (owner && i < n) actions[i] = uint8_t(a >> 31);
  }
}

}  // namespace

// Tiles per wave, by the batch's size: one tile while that makes at most
// three waves per SIMD (1,024 SIMDs), since a wave alone on its SIMD waits
// out its own instruction stream, which a tile takes a fourth of (64 steps of
// 10,007 environments: four tiles 228 us, two 123, one 75; of 49,152:
// 228, 200, 170); two tiles up to 131,072 (65,536: 228, 200, one tile 216;
// 131,072: four 369, two 364); above, four, which repeat no dynamics (262,144:
// 683, two 715).  A block stages the weights and gathers its fragments before
// its first step, so short rollouts take one tile only up to 8,192 environments
// per step (one step of 49,152: one tile 15.9 us, two 11.7; of 16,384: 9.4 and
// 8.4; of 4,096: 7.0 and 7.3; two steps of 24,576: 12.2 and 11.3; four of
// 32,768: 16.0 and 15.9).
constexpr uint32_t kOneTileMaxEnvs = 49152, kTwoTilesMaxEnvs = 131072;
constexpr uint32_t kOneTileEnvsPerStep = 8192;

template <int kTiles>
static void actions_as(const float *obs, uint32_t n, const uint16_t *policy_w, uint8_t *actions,
                       hipStream_t stream) {
  // The same number of rounds for every block, as few blocks as fit the GPU
  // at once (four waves per SIMD): a block that came later would stage the
  // weights again for one round.
  constexpr uint32_t kEnvs = kResidentWaves * MlpPolicy<kTiles>::kEnvsPerWave, kMost = 1024;
  const uint32_t work = (n + kEnvs - 1u) / kEnvs, rounds = (work + kMost - 1u) / kMost;
  hipLaunchKernelGGL(k_policy_actions<kTiles>, dim3((work + rounds - 1u) / rounds),
                     dim3(kResidentBlock), 0, stream, obs, n, policy_w, actions);
}

hipError_t launch_policy_actions(const float *obs, uint32_t n, const uint16_t *policy_w,
                                 uint8_t *actions, hipStream_t stream) {
  if (n <= kOneTileMaxEnvs) actions_as<1>(obs, n, policy_w, actions, stream);
  else if (n <= kTwoTilesMaxEnvs) actions_as<2>(obs, n, policy_w, actions, stream);
  else actions_as<4>(obs, n, policy_w, actions, stream);
  return hipGetLastError();
}

template <int kTiles>
static void policy_as(const RolloutParams &p, hipStream_t stream) {
  constexpr uint32_t kEnvs = kResidentWaves * MlpPolicy<kTiles>::kEnvsPerWave;
  const dim3 grid((p.n + kEnvs - 1u) / kEnvs), b(kResidentBlock);
  switch (traj_kind(p, sizeof(float))) {
    case Traj::kNone:
      hipLaunchKernelGGL((k_resident_policy<Traj::kNone, kTiles>), grid, b, 0, stream, p);
      break;
    case Traj::kAny:
      hipLaunchKernelGGL((k_resident_policy<Traj::kAny, kTiles>), grid, b, 0, stream, p);
      break;
    default:
      hipLaunchKernelGGL((k_resident_policy<Traj::kAll, kTiles>), grid, b, 0, stream, p);
      break;
  }
}

hipError_t launch_resident_policy(const RolloutParams &p, hipStream_t stream) {
  if (p.n <= kOneTileMaxEnvs && p.n <= uint64_t(kOneTileEnvsPerStep) * p.T) policy_as<1>(p, stream);
  else if (p.n <= kTwoTilesMaxEnvs) policy_as<2>(p, stream);
  else policy_as<4>(p, stream);
  return hipGetLastError();
}

}  // namespace cp

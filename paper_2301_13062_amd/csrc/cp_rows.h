// cp_rows.h -- how a whole-rollout launch stores a trajectory whose rows start
// off the 128-byte lines (cp_resident.h): by rows, and in which blocks, or by
// waves.  Host code without HIP.
//
// Every wave that stores its own values leaves parts of two lines per row, which
// another wave completes at another time.  By rows (RowStage) a block stores its
// piece of each row in whole lines, a barrier and a pass through LDS per step;
// by waves the blocks of one XCD lie next to each other, so that most parts of
// lines meet in its L2.  Times below are of fresh allocations, two trajectories
// in turn.
#pragma once

#include <stdint.h>

namespace cp {

// Whether every row of obs and of reward starts on a 128-byte line.  The flags'
// rows do not count (4,194,240 x 64: 1,189 us by waves, 1,180 by rows).
inline bool rows_on_lines(uint32_t n, uint32_t elem, uintptr_t obs, uintptr_t reward) {
  return (obs | reward | uintptr_t(n * uint64_t(elem < 4 ? elem : 4))) % 128u == 0u;
}

// By rows pays where the 256 MB memory-side cache does not absorb the
// trajectory (as it does up to there: 200,003 x 64 in binary32, 269 MB: 55 us by
// waves, 75 by rows) and the row blocks fill the CUs: a block's step takes 0.74
// us however few blocks there are, where by waves it takes the batch's share of
// the bandwidth.  binary32 (4,097 x 5,230 1.39 ms by waves, 3.80 by rows;
// 50,001 x 952 266 us and 695; 100,001 x 476 279 and 353; 120,001 x 178 112 and
// 136; 131,071 x 163 131 and 127, x 908 779 and 683) needs a block on every CU,
// binary64 (50,001 x 540 221 and 443; 90,001 x 210 179 and 181; 120,001 x 225
// 245 and 198) on most.
constexpr uint64_t kRowsMinBytes = uint64_t(384) << 20;
constexpr uint32_t kComputeUnits = 256, kRowsMinEnvs32 = 128000;
// Blocks of 1,024, and below this size, where those leave CUs idle or with
// twice the work of others, of 512 (300,007 x 64: 146 and 105 us; 500,009:
// 152 and 168).
constexpr uint32_t kRowsWideMinEnvs = 400000;
// The rounds of one block per CU have to be three quarters full (binary32,
// 150,001 x 222, 293 blocks: 200 us by waves, 226 by rows; 180,001 x 264, 352:
// 273 and 269; 200,003 x 238, 391: 307 and 252; binary64, 150,001 x 126 179 and
// 203, 180,001 x 150 247 and 259, 200,003 x 135 260 and 237).
// In binary16 a CU holds one row block, of 2,048 environments, at a time, and
// the waves of the other form keep together besides: rows gain from 1,000,000
// environments on, where their rounds are nearly full and the trajectory is
// long (1,000,003 x 115 420 us by waves, 397 by rows; 3,000,001 x 38 465 and
// 433, of 64 743 and 676; but 1,100,001 x 69 328 and 363; 3,200,001 x 24 337
// and 348; 3,000,001 x 17 231 and 239; 850,001 x 135 420 and 456; 200,003 x
// 384 240 and 614).
constexpr uint64_t kRowsMinBytes16 = uint64_t(800) << 20;
constexpr uint32_t kRowsMinEnvs16 = 1000000, kRowsBlockEnvs16 = 2048;

// Threads per block of the rows kernel for a launch of T steps of n
// environments whose state elements have `elem` bytes, or 0: by waves.
inline uint32_t rows_block(uint32_t n, uint64_t T, uint32_t elem, uintptr_t obs, uintptr_t reward) {
  if (rows_on_lines(n, elem, obs, reward)) return 0u;
  const bool half = elem == 2u;
  const uint32_t threads = half || n >= kRowsWideMinEnvs ? 1024u : 512u;
  const uint32_t envs = half ? kRowsBlockEnvs16 : threads;
  const uint64_t blocks = (n + uint64_t(envs) - 1u) / envs;
  const uint64_t slots = (blocks + kComputeUnits - 1u) / kComputeUnits * kComputeUnits;
  const bool full = half ? 16u * blocks >= 15u * slots : 4u * blocks >= 3u * slots;
  const uint32_t least = half ? kRowsMinEnvs16 : elem == 4u ? kRowsMinEnvs32 : 0u;
  const bool large = n * T * (4u * elem + 5u) >= (half ? kRowsMinBytes16 : kRowsMinBytes);
  return full && large && n >= least ? threads : 0u;
}

}  // namespace cp

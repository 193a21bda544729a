// Dispatch rules by size, free of device calls (the CPU tests check them): which
// of two forms of a kernel a call takes.
#pragma once

#include <algorithm>
#include <cstdint>

namespace cdd {

// Compute units of the MI355X.
constexpr int64_t kComputeUnits = 256;

// Whether the workgroups of a batch of DM trials take two neighbouring blocks of a
// channel each, which share the table of chirp phases, or one.  An odd count of
// blocks leaves a spare group that repeats the last block: two are taken as long as
// the blocks transformed per block of work (`doubled` / `blocks`: nchan 2 ceil(n/2)
// and nchan n, summed over the beams) stay below what sharing gains at this length
// and count of trials per block.  Measured on a full card (512 to 2048 channels), time with
// two over time with one:
//   trials              3            16           48
//   blocks/channel    1    3   32   1    3   33   1    3    5   33
//    512 points     1.00 0.76 0.86 1.03 0.90 1.01 1.12 1.10 1.13 0.96
//   1024 points     1.00 0.81 0.78 1.11 1.05 0.92 1.22 1.12 1.08 0.95
//   2048 points     1.05 0.98 0.78 1.19 1.13 0.95 1.24 1.17 1.03 0.97
//   4096 points     0.96 0.94 0.75 1.08 1.06 0.86 1.10 1.08 0.95 0.86
// While every block can have a compute unit to itself, one per workgroup is the
// faster form (16 channels: 1.00 to 1.12 at 512 points, 1.07 with 48 trials at
// 2048), but for a few trials at 4096 points (0.96).
inline bool two_blocks_pay(int N, double trials, int64_t blocks, int64_t doubled) {
  if (N > 2048 && trials <= 4.0) return true;
  if (blocks <= kComputeUnits) return false;
  double limit = N <= 512    ? (trials <= 16.0 ? 4.0 / 3.0 : 1.04)
                 : N <= 1024 ? 1.09 + 2.0 / trials
                 : N <= 2048 ? 1.09 + 1.0 / trials
                             : 1.19 + 1.0 / trials;
  limit = std::min(limit, 4.0 / 3.0);
  return (double)doubled <= limit * (double)blocks * (1.0 + 1e-12);
}

}  // namespace cdd

// Dispatch rules by size, free of device calls (the CPU tests check them): which
// of two forms of a kernel a call takes.
#pragma once

#include <algorithm>
#include <cmath>
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

// Units of work that one value of the batch kernel's counter stands for, per beam of
// a launch (listed longest unit first; points: transformed per unit, all trials).
// The counter hands out one value per 12 ns, which set the pace of short units (256
// points, 2 trials, 512 channels x 250,000 samples: 250,000 units, 3.05 ms per pass);
// a unit takes about 1.1 ns per point.  So many are taken that the counter is asked
// for half the values it can give (22 points per resident workgroup and value), as
// long as each workgroup comes back four times from there to the end of the launch,
// which keeps the end even: that pass 1.20 ms, 4 trials at 512 points 2.16 -> 1.34,
// 2 at 1024 points 1.03 -> 0.76.  Units of 64 trials are taken singly, also beside
// beams of many short units.
inline void units_per_value(int n, const double* points, const int64_t* units, int64_t resident,
                            int32_t* take) {
  int64_t left = 0;
  for (int i = 0; i < n; ++i) left += units[i];
  const int64_t grid = std::max<int64_t>(1, std::min(left, resident));
  for (int i = 0; i < n; ++i) {
    const double want = std::ceil(22.0 * (double)grid / std::max(1.0, points[i]));
    take[i] = (int32_t)std::max(1.0, std::min({want, 16.0, (double)(left / (4 * grid))}));
    left -= units[i];
  }
}

// Whether the incoherent path detects straight from the time-major record or from
// a channel-major copy.  A thread of the direct form adds up the n_int samples of
// its 4 outputs (8 where it has one channel) in turn, a serial chain that lasts as
// long for a small record as for a large one; the copy costs its bytes and two
// launches.  A call on new inputs (us), copy -> direct:
//                        n_int 16     24            32            64
//   8 bits  16 x 4,000   19 -> 14     19 -> 20      19 -> 25      19 -> 42
//           16 x 40,000  19 -> 16     19 -> 21      19 -> 27      23 -> 47
//           64 x 40,000  24 -> 16     22 -> 21      26 -> 25      28 -> 46
//           2 x 400,000  25 -> 18     25 -> 20      26 -> 20      31 -> 40
//          16 x 400,000  64 -> 19     62 -> 25      66 -> 30      75 -> 54
//   float   16 x 4,000   19 -> 15     19 -> 21      19 -> 26      19 -> 47
//           64 x 40,000  35 -> 24     33 -> 31      32 -> 39      32 -> 68
//           2 x 400,000  47 -> 21     53 -> 27      54 -> 29      59 -> 50
//          512 x 40,000 346 -> 39    399 -> 43     359 -> 52     370 -> 79
//          128 x 4,000   20 -> 23     20 -> 31      21 -> 35      24 -> 68
// With fewer than 32 outputs the chain is shorter (500 samples, n_int 48: 19 -> 16).
inline bool detect_from_record(bool float_samples, int64_t nchan, int64_t nsamp, int n_int) {
  if (nchan < 2 || n_int > 64) return false;
  // the chain, against the time of the copy's launches
  const int64_t rounds = std::min<int64_t>(4, (nsamp / n_int + 7) / 8);
  const int64_t chain = rounds < 4      ? 96
                        : float_samples ? (nchan <= 4 ? 72 : nchan < 100 ? 64 : 48)
                                        : (nchan <= 256 ? 80 : 64);
  if (n_int * rounds <= chain) return true;
  // else the record must be large enough for the copy's bytes to outlast the chain
  const int64_t samples = nchan * nsamp;
  if (n_int > 32) return samples >= 6000000 || (float_samples && nsamp >= 200000);
  return samples >= (n_int <= 20 ? 1500000 : 3000000) || nsamp >= 200000;
}

// Threads per phase bin of a fold (each takes every so many-th period): a workgroup
// while the bins do not fill the card by themselves, then a wave; a thread with more
// bins than resident waves, or with a few periods only, which leave a wave's lanes
// idle.  1,000,000 samples (us), thread -> wave:
//   periods      1           2           3           4
//   1025 bins  248 -> 353  226 -> 179  220 -> 121  222 -> 90
//   4096 bins   56 -> 123   56 -> 62    56 -> 42    58 -> 32
//   8192 bins   30 -> 99    30 -> 51    30 -> 36    31 -> 28
inline int fold_threads(int64_t t_int, double period, int nbins) {
  if (nbins <= 1024) return 256;
  const int least = 2 + (nbins > 2048) + (nbins > 4096);
  return nbins <= 8192 && (double)t_int >= least * period ? 64 : 1;
}

}  // namespace cdd

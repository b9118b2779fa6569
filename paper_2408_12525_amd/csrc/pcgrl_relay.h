// Whether, and in which shape, a pcgrl_rollout runs as a relay of wavefronts.  Plain C++, apart from the
// kernel, so that the rule can be called on the host for batches and kernels of any size.
#pragma once
#include <cstdint>

namespace pcgrl {

constexpr int kRelaySteps = 8;  // steps that a relay's wavefronts hand on to each other at a time (see rollout_relay_kernel)

// Searchers, and observers that take the steps in turn; no searchers: not as a relay.
struct RelayShape {
  int searchers, turns;
};
struct RelayCase {
  int rows;                                // of the size class
  bool binary;                             // the binary problem
  int per_simd;                            // wavefronts of the relay's kernel that the registers of a SIMD hold
  int compute_units;
  int64_t workgroups;
  int observers;                           // that one step's observations take in a workgroup
  int64_t obs_bytes, step_bytes;           // of one level's observation, and of all in a step
  int64_t lds_tables, lds_observer;        // bytes of a workgroup, and more for every observer
  int64_t steps, slots;                    // of the rollout
};

// A relay shares a chain of one wavefront per step out among several, at the price of following the
// levels in each: it pays while the wavefronts have the SIMDs mostly to themselves, which is a question of
// workgroups per compute unit, and while it is not the stores that the rollout waits for.  Measured with
// 31-cell windows, us a step of 32-step rollouts: without / 4 searchers and 4 observers / 4 and 2 / 2 and 2 /
// 2 and 1; the levels are as many workgroups, and (w) says how many wavefronts a SIMD holds by registers:
//            16x16 binary (7)                 32x32 binary (7)                 64x64 binary (7)
//    64   1.39 / 0.87 / 0.91 / 1.05 / 1.24   1.38 / 0.96 / 0.99 / 0.99 / 1.15   1.11 / 0.82 / 0.88 / 0.90 / 1.04
//   512   1.82 / 1.15 / 1.13 / 1.29 / 1.44   2.02 / 1.34 / 1.30 / 1.45 / 1.55   1.41 / 1.17 / 1.18 / 1.15 / 1.27
//   768   1.95 / 1.66 / 1.29 / 1.45 / 1.54   1.99 / 1.71 / 1.47 / 1.56 / 1.65   1.50 / 1.70 / 1.36 / 1.29 / 1.39
//  1024   1.97 / 2.20 / 1.81 / 1.96 / 1.64   2.14 / 2.27 / 1.91 / 1.98 / 1.80   1.65 / 2.26 / 1.81 / 1.79 / 1.58
//  1280   2.14 / 2.47 / 2.05 / 2.21 / 2.49   2.32 / 2.48 / 2.05 / 2.19 / 2.26   1.70 / 2.49 / 2.08 / 2.04 / 2.16
//  1536   2.22 / 2.92 / 2.39 / 2.61 / 2.75   2.29 / 2.89 / 2.31 / 2.44 / 2.59   1.88 / 3.00 / 2.35 / 2.40 / 2.43
//            16x16 maze (5)                   32x32 maze (6)                   64x64 maze (7)
//    64   1.02 / 0.67 / 0.85 / 0.85 / 1.28   1.12 / 0.66 / 0.79 / 0.79 / 1.15   1.23 / 0.78 / 0.89 / 0.92 / 1.22
//   512   1.19 / 1.25 / 1.03 / 1.01 / 1.40   1.30 / 0.90 / 0.98 / 0.97 / 1.25   1.45 / 1.07 / 1.13 / 1.15 / 1.37
//   768   1.35 / 1.79 / 1.70 / 1.75 / 1.48   1.46 / 1.31 / 1.11 / 1.10 / 1.34   1.64 / 1.57 / 1.31 / 1.31 / 1.49
//  1024   1.37 / 2.31 / 1.85 / 1.93 / 2.58   1.49 / 1.94 / 1.59 / 1.58 / 1.43   1.67 / 2.27 / 1.82 / 1.83 / 1.59
//            16x16 dungeon (5)                32x32 dungeon (5)                64x64 dungeon (6)
//    64   1.28 / 0.80 / 1.05 / 1.04 / 1.63   1.39 / 0.76 / 0.97 / 0.95 / 1.44   1.52 / 0.91 / 1.07 / 1.10 / 1.53
//   512   1.46 / 1.46 / 1.25 / 1.21 / 1.75   1.56 / 1.39 / 1.18 / 1.13 / 1.54   1.75 / 1.23 / 1.36 / 1.35 / 1.66
//   768   1.66 / 2.09 / 2.06 / 2.08 / 1.82   1.75 / 1.98 / 1.88 / 1.86 / 1.65   2.00 / 1.80 / 1.57 / 1.55 / 1.81
//  1024   1.68 / 2.71 / 2.27 / 2.35 / 3.25   1.81 / 2.57 / 2.12 / 2.17 / 2.81   2.06 / 2.65 / 2.17 / 2.17 / 1.96
// (2048 32-row levels are 1024 workgroups of two: binary 2.52 / - / 2.19 / 2.35 / 2.10, maze 2.52 / - / 2.22 / 2.18 / 1.91.)
inline RelayShape relay_shape(const RelayCase& c) {
  constexpr RelayShape kNone = {0, 0};
  const int64_t per_cu = (c.workgroups + c.compute_units - 1) / c.compute_units;
  const bool small_binary = c.binary && c.rows < 64;
  // Within one piece leader, searchers, observers and adder run one after the other, and only the long searches of
  // small binary levels make up for that at once.  Without / with a relay: one step 5.7 / 6.0 us (64 16x16 binary
  // levels) to 4.2 / 5.0 (16x16 maze); two steps 3.7 / 3.4 and 2.7 / 2.9; three 3.0 / 2.5, 2.1 / 2.1; eight steps of 512
  // 16x16 maze levels 1.73 / 1.79, twelve 1.53 / 1.39; eight of 1024 64x64 binary ones 2.34 / 2.50.
  const int fewest = small_binary ? 2 : per_cu > 3 || (per_cu > 1 && c.rows == 16) ? kRelaySteps + 1 : 3;
  if (c.steps < fewest) return kNone;
  // 63-cell windows: 768 16x16 binary levels (9.1 MB a step) 2.29 / 1.74 us, 512 32x32 maze levels (10.2) 2.00 / 1.95,
  // 600 (11.9) 2.52 / 2.72, 512 dungeon levels (16.3) 3.17 / 3.38, 2048 16x16 binary levels (24) 4.8 / 5.4.
  if (c.step_bytes > ((int64_t)11 << 20)) return kNone;
  RelayShape s = kNone;
  if (per_cu <= 1) s = {4, 4};
  else if (per_cu == 2 && c.per_simd >= 6) s = {4, 4};
  // (9-cell windows, 4 and 2 / 2 and 2: 512 32x32 dungeons 0.91 / 0.96; 63 cells: 512 16x16 maze levels 1.91 / 2.08 without / with)
  else if (per_cu == 2 && c.obs_bytes <= 16384) s = {c.obs_bytes < 2048 ? 4 : 2, 2};
  else if (c.per_simd < 6) return kNone;
  else if (per_cu == 3) s = {4, 2};
  else if (per_cu == 4 && c.obs_bytes <= 8192) s = {2, 1};
  // (not all at once on the machine any more, and still ahead with small windows: 45 cells 2.21 / 2.32)
  else if (per_cu == 5 && small_binary && c.obs_bytes <= 4096) s = {4, 2};
  else return kNone;
  while (s.turns * c.observers > 4) s.turns /= 2;
  // Wavefronts that take turns are not ordered among each other: a slot that is written more than once in
  // the rollout must be written by the same wavefront every time, i.e. the number of turns has to divide
  // the number of slots.
  if (c.slots != c.steps)
    while (s.turns > 1 && c.slots % s.turns != 0) s.turns /= 2;
  if (s.turns < 1) return kNone;
  // One observer follows the levels and builds every observation, as without a relay, and the longer it is at
  // that the less there is to gain: with one slot 64 16x16 binary levels 1.44 / 1.21 us, 512 32x32 dungeons
  // 1.64 / 1.50, with a 63-cell window 64 16x16 binary levels 2.24 / 2.10, 64x64 maze levels 2.54 / 2.40, but 512 64x64
  // binary levels (12 KB an observation) 1.82 / 1.92, dungeons (32 KB) 3.57 / 3.68.
  if (s.turns == 1 && (per_cu > 4 || (c.rows == 64 && c.obs_bytes > (c.binary ? 8 : 24) * 1024))) return kNone;
  // (a workgroup of at most 64 KB, and all those of a compute unit within its 160 KB)
  const int64_t lds = c.lds_tables + c.lds_observer * c.observers * s.turns;
  if (lds > 64 * 1024 || per_cu * lds > 160 * 1024) return kNone;
  return s;
}

}  // namespace pcgrl

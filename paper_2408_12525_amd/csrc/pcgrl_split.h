// Whether a step or a rollout runs as one wavefront a level group, or as a metrics wavefront and observation
// wavefronts.  Plain C++, apart from the kernels, so that the rules can be called on the host for any size.
#pragma once
#include <cstddef>
#include <cstdint>

#include "../../include/pcgrl.h"

namespace pcgrl {

// How observations are stored: ordinary, non-temporal and write-through stores.
enum : int { kStoreCached = 0, kStoreStream = 1, kStoreThrough = 2 };
// Where a rollout's ring of observation slots goes: ordinary stores into one that stays in the memory-side cache of 256 MB,
// into one that is somewhat larger, and into a much larger one; other stores.  (Of 64-row levels, 8 slots of 27 MB, two wavefronts
// take 1.04 times as many a second as one into 219 MB, and 0.95 times as many into 220.)
enum : int { kRingFits = 0, kRingSpills = 1, kRingBeyond = 2, kRingStreams = 3 };
constexpr int ring_of(int store, int64_t ring_bytes) {
  return store != kStoreCached ? kRingStreams : ring_bytes <= (int64_t)219 << 20 ? kRingFits : ring_bytes <= (int64_t)448 << 20 ? kRingSpills : kRingBeyond;
}

// Results never depend on a launch shape; every row below is a measurement on MI355X (per-step launches replayed
// from a HIP graph, rollouts of 8 to 100 steps).  A table is read top down and the first row whose conditions all
// hold decides; ranges are inclusive.
constexpr int64_t kMax = INT64_MAX;
constexpr int64_t kMB = (int64_t)1 << 20;
// (each with whole 128-byte lines to a level's observation, and sixteen times that without)
enum : int { kCached = 17 << kStoreCached, kStream = 17 << kStoreStream, kThrough = 17 << kStoreThrough, kAnyStore = 255, kNoLines = 240 };
enum : int { kSpills = 17 << kRingSpills, kBeyond = 17 << kRingBeyond };
struct SplitRule {
  int S;                            // size class (16 / 32 / 64 rows), 0 = any
  int64_t batch_lo, batch_hi;       // environments
  int64_t obs_lo, obs_hi;           // bytes of one level's observation
  int64_t step_lo, step_hi;         // bytes of one step's observations, whole batch
  int problem;                      // -1 = any
  int stores;                       // the ways of storing, or rings, that it holds for
  int split;                        // 1: a metrics wavefront and observation wavefronts per workgroup
};
struct SplitCase {
  int S, problem;
  int64_t batch, obs_bytes, step_bytes;
  bool whole_lines;                 // a multiple of 128 bytes from one level's observation to the next
};

// pcgrl_step.  Two wavefronts per level group shorten the dependent chain of a launch at the price
// of loading the level twice.
inline constexpr SplitRule kStepSplit[] = {
    {16, 1, 8192, 0, kMax, 0, kMax, -1, kAnyStore, 1},           // -10...-25 % per step at batches of 512...8192
    {16, 8193, kMax, 3072, kMax, 256 * kMB + 1, 448 * kMB, -1, kAnyStore, 0},  // stored through the cache: +17 %
    {16, 8193, 12288, 0, kMax, 0, kMax, -1, kAnyStore, 1},       // us one / two at 8193, 12 288, 20 000: binary (15 cells) 7.7 / 7.4, 8.3 / 8.2, 10.0 / 10.1, maze (15)
                                                      // 6.3 / 5.6, 7.0 / 6.5, 8.5 / 8.6, dungeon (7) 6.4 / 5.9, 7.2 / 6.9, 8.8 / 9.0
    {16, 8193, kMax, 1536, kMax, 0, kMax, -1, kAnyStore, 1},     // maze16 -13 % at 12 288, -2...-4 % from 32 768; binary16 -3 % at 262 144
    {32, 1, 4096, 0, kMax, 0, kMax, -1, kAnyStore, 1},           // dungeon32 -16 % at 256, -7 % at 4096
    {32, 4097, 4608, 0, kMax, 0, kMax, -1, kAnyStore, 1},        // us one / two at 4097: maze 6.18 / 5.96 (9 cells), binary 8.61 / 8.45, dungeon 6.84 / 6.54
    {32, 4609, 6144, 1024, kMax, 0, kMax, -1, kAnyStore, 1},     // at 5000 and 6000: maze (15 cells) 6.93 / 6.79, 7.24 / 7.08, (21) 7.30 / 6.91, 7.61 / 7.23; with
                                                      // 9 cells dungeon 7.26 / 7.33, 7.64 / 7.64
    {32, 4097, 16384, 2560, kMax, 0, kMax, -1, kAnyStore, 1},    // us one / two, observation: maze 8192 10.2 / 9.7 (4.8 KB), 7.8 / 7.9 (2.2 KB),
                                                      // 16 384 17.2 / 16.3, 11.9 / 12.3; dungeon 16 384 14.3 / 13.6 (3.5 KB); binary 8192 11.0 / 10.6 (2.9 KB)
    // Larger batches by how they store, us one / two with a buffer for each step (whole lines), and what one is of two where a
    // single buffer is written through.  From 128 MB a step on, observations of 3 KB and more go through the cache if they have
    // a buffer for each step: dungeon (21 cells, 143 MB) 40 000 31.8 / 36.0, (23) 32 768 0.96, maze (25) 50 000 0.79, but maze
    // (31 cells, 159 MB) 32 768 32.1 / 30.7, dungeon (25) 1.01.  Beyond 168 MB none was ahead.
    {32, 16385, kMax, 2560, 3071, 0, 168 * kMB, PCGRL_BINARY, kStream | kThrough, 1},  // 31 cells 16 385 16.3 / 15.5, 1.04, 50 000 31.3 / 29.1, 1.00
    {32, 16385, kMax, 2560, 3071, 0, 168 * kMB, PCGRL_MAZE, kStream, 1},  // 23 cells 16 385 12.0 / 11.9, 1.02, 32 768 19.1 / 18.7, 0.94, 50 000 27.0 / 26.3, 0.93
    {32, 16385, kMax, 2816, 3071, 0, 168 * kMB, PCGRL_DUNGEON, kStream & kNoLines, 1},  // 19 cells 16 385 1.04, 24 001 19.1 / 17.8, 40 000 28.8 / 26.0, but whole lines
                                                      // 24 001 0.98, 32 768 20.0 / 21.1, one buffer 0.94; 18 cells 32 768 0.93
    {32, 16385, kMax, 3072, 3327, 0, 168 * kMB, PCGRL_DUNGEON, kThrough, 0},  // 20 cells 24 001 0.98, 40 000 0.96; with a buffer for each step 1.03, 1.04
    {32, 16385, kMax, 3072, kMax, 0, 168 * kMB, -1, kStream | kThrough, 1},  // maze (25 cells) 28 000 1.13, 1.00, (31) 16 385 17.0 / 16.0, 1.07, 24 001 23.5 / 22.3, 1.06,
                                                      // dungeon (21) 24 001 18.5 / 17.2, 1.01, 32 768 23.6 / 22.0, 1.00, (25) 24 001 24.9 / 23.9, 1.05, binary (41) 32 768 35.9 / 33.9
    {32, 16385, kMax, 4096, 4607, 0, 168 * kMB, -1, kCached & kNoLines, 1},  // maze (29 cells) 32 768 32.5 / 31.3, 40 000 38.9 / 37.4, whole lines 0.95, 0.94; dungeon (23) 1.00
    {32, 16385, kMax, 4608, kMax, 0, 168 * kMB, -1, kCached, 1},
    {64, 1, 4096, 0, kMax, 0, kMax, -1, kAnyStore, 1},           // maze64 -12 % at 256, -4 % at 4096; none from 8192 on
    {64, 4097, 12288, 6000, kMax, 0, kMax, -1, kAnyStore, 1},    // dungeon (7.7 KB) 4097 10.5 / 10.1, 8192 16.0 / 15.0, 12 288 20.7 / 19.5, binary (6.1 KB)
                                                      // 10.3 / 9.9, 13.5 / 13.4, 17.4 / 16.8; maze (4.8 KB) 8.8 / 8.6, 12.1 / 12.3, 15.0 / 15.7
    {0, 1, kMax, 0, kMax, 0, kMax, -1, kAnyStore, 0},
};
// pcgrl_rollout (each wavefront keeps its own copy of the level for all the steps).
inline constexpr SplitRule kRolloutSplit[] = {
    {16, 1, 2048, 0, kMax, 0, kMax, -1, kAnyStore, 1},           // -35 % per step at 64 and 1024
    {16, 2049, 12288, 0, 4095, 0, kMax, -1, kAnyStore, 1},       // binary16 +39 % steps/s at 4096, +22 % at 8192
    {16, 12289, kMax, 1536, 4095, 0, kMax, -1, kAnyStore, 1},    // binary16 -5...-9 % per step from 16 384 to 131 072
    {16, 2049, 4096, 4096, kMax, 0, kMax, -1, kAnyStore, 1},     // maze16 -20 % at 4096
    {16, 16384, kMax, 4096, kMax, 0, kMax, -1, kAnyStore, 1},    // maze16 -2...-3 % (at 8192: +6 %, hence the gap)
    {32, 1, 4096, 0, kMax, 0, kMax, -1, kAnyStore, 1},           // -43 % at 256, -24 % at 4096
    {16, 12289, 65536, 0, 1535, 0, kMax, PCGRL_BINARY, kAnyStore, 1},  // us a step one / two at 20 000, 40 000: 7 cells 6.4 / 6.2, 9.8 / 9.5, 15 cells 6.6 / 6.4, 10.8 / 10.2;
                                                      // 200 001 (9) 38.8 / 40.2; others no gain (maze, 9 cells, 20 001 4.3 / 4.4)
    {32, 4097, 5120, 4608, 5999, 0, kMax, PCGRL_DUNGEON, kBeyond, 0},  // 25 cells, one of two, 48 slots (1 GB) 4097 0.95...0.96, 5120 0.94...0.97; 16 slots 1.02...1.06, 8 slots 1.17...1.23
    {32, 4353, 5120, 3840, 4607, 0, kMax, PCGRL_DUNGEON, kBeyond, 0},  // 23 cells, 48 slots 4097 1.03, 4608 0.96...0.97, 5120 0.94...0.96; 8 slots 1.09...1.12
    {32, 4097, 5120, 0, 5999, 0, kMax, -1, kAnyStore, 1},        // at 4097: maze (15) 3.5 / 3.0, dungeon (15) 4.0 / 3.4; at 6000 4.0 / 3.9, 4.7 / 4.8; dungeon (31) 4200 6.9 / 7.0
    {32, 10240, 131072, 0, 5999, 0, kMax, PCGRL_MAZE, kAnyStore, 1},  // 15 cells at 8192, 12 288, 20 000 4.7 / 4.7, 6.5 / 6.0, 9.3 / 8.7, 120 000 1.02, 31 cells 7.0 / 7.2, 12.5 / 11.6,
                                                      // 19.6 / 18.6, 70 000 1.00...1.02; 45 cells 10 240 to 70 000 0.98...1.01
    {32, 10240, 12800, 0, 8191, 0, kMax, PCGRL_DUNGEON, kAnyStore, 1},  // 15 cells 5.5 / 5.6, 7.8 / 7.5, (14 001) 8.7 / 8.9, 23 cells 6.4 / 6.5, 11.5 / 10.6, 18.0 / 17.5, 31 cells 1.01...1.04
    {32, 4097, kMax, 0, kMax, 0, kMax, PCGRL_BINARY, kAnyStore, 1},  // +10 % steps/s at 16 384 (dungeon: +-2 %)
    {64, 1, 8192, 0, kMax, 0, kMax, -1, kAnyStore, 1},           // -6 %
    {64, 8193, kMax, 0, 2047, 32 * kMB + 1, kMax, PCGRL_DUNGEON, kSpills, 0},  // one of two: 15 cells, 8 slots at 20 000 (34 MB a step) 0.98, 24 001 0.95...1.01, 13 cells at 32 768 0.96
    {64, 8193, 32768, 0, 2047, 0, kMax, PCGRL_DUNGEON, kAnyStore, 1},  // 15 cells at 8193, 10 000, 16 000 8.2 / 7.5, 9.5 / 9.0, 13.9 / 13.4, at 32 768 1.03...1.06; 14 cells, 16 slots at 10 887 9.1 / 8.5
    {64, 8193, kMax, 0, 2047, 16 * kMB + 1, kMax, -1, kSpills, 0},  // one of two, 8 slots: maze (20 cells) 24 001 0.88, (15) 32 768 0.95, binary (20) 24 001 0.95, (25) 20 000 0.88;
                                                      // 16 slots: maze (20) 12 000 0.95; 48 slots of up to 9 MB are ahead as in the next row
    {64, 8193, 24576, 0, 2047, 0, kMax, -1, kAnyStore, 1},       // 15 cells at 8193, 10 000, 16 000, 24 001: binary 6.4 / 6.1, 6.8 / 6.5, 10.1 / 9.9, 13.3 / 13.3 (48 slots 1.01), maze 6.8 / 6.3,
                                                      // 7.8 / 7.4, 11.0 / 10.6, 15.3 / 15.2 (1.03); 32 768 0.95...1.01
    {64, 8193, 12288, 6000, kMax, 0, kMax, PCGRL_DUNGEON, kAnyStore, 1},  // 31 cells 13.8 / 12.8, 16.4 / 15.5, 19.1 / 18.5; 23 cells 10.1 / 10.1, 11.4 / 11.9; 41 cells, 48 slots 0.98...1.00
    {0, 1, kMax, 0, kMax, 0, kMax, -1, kAnyStore, 0},
};

template <size_t N>
constexpr int first_match(const SplitRule (&table)[N], const SplitCase& c, int how) {
  for (const SplitRule& r : table)
    if ((r.S == 0 || r.S == c.S) && c.batch >= r.batch_lo && c.batch <= r.batch_hi && c.obs_bytes >= r.obs_lo &&
        c.obs_bytes <= r.obs_hi && c.step_bytes >= r.step_lo && c.step_bytes <= r.step_hi && (r.problem < 0 || r.problem == c.problem) &&
        ((r.stores >> (how + (c.whole_lines ? 0 : 4))) & 1) != 0)
      return r.split;
  return 0;
}
constexpr int split_step(const SplitCase& c, int store) { return first_match(kStepSplit, c, store); }
constexpr int split_rollout(const SplitCase& c, int ring) { return first_match(kRolloutSplit, c, ring); }

}  // namespace pcgrl

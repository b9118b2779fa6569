// Whether, and into how many spans, a pcgrl_rollout is cut up along its steps.  Plain C++, apart from the
// kernels, so that the rule can be called on the host for batches and rollouts of any size.
#pragma once
#include <algorithm>
#include <cstdint>

#include "../../include/pcgrl.h"

namespace pcgrl {

struct SpanCase {
  int rows;                // of the size class
  int problem;             // PCGRL_BINARY / MAZE / DUNGEON
  bool observed;           // with observations, a slot for every step
  int64_t batch, steps;    // levels, steps of the rollout
  int64_t cells, max_w;    // of a level, half way between the mean and the largest shape; the width of the largest
  int64_t obs_bytes;       // of one level's observation
  int64_t window_bits;     // its cells times channels
  int64_t step_bytes;      // of the observations of a step
  int64_t episode;         // steps that an episode has at the least; 0: a level never starts again
};
struct SpanShape {
  int spans, steps;  // of the rollout, and of a span; one span: not cut up
};

// As many spans as give this many levels to take through their steps side by side.  Every span begins with
// the metrics from scratch, which cost about as much as four of its steps on 16 rows and eight on 64, so that
// the machine should be full and not much more.  Us for a rollout with 31-cell windows, 1024 / 2048 / 4096 / 8192 /
// 16 384 levels side by side:
//   64 levels, 128 steps   16x16 binary 31.9 / 26.8 / 22.8 / 25.0     32x32 30.2 / 24.3 / 25.3 / 31.4   64x64 29.8 / 28.8 / 34.3 / 48.4
//   512 levels, 64 steps   16x16 maze   82.6 / 47.5 / 31.1 / 31.3 / 33.2   32x32 58.2 / 37.9 / 34.2 / 37.6 / 42.5   64x64 59.7 / 49.0 / 50.4 / 57.7 / 75.8
//   1024 levels, 32 steps  16x16 binary    - / 55.9 / 36.9 / 32.8 / 33.5   32x32 - / 64.4 / 53.1 / 41.8 / 46.5      64x64 - / 49.7 / 45.5 / 49.7 / 65.9
// A level is cut into kMostSpans at the most, however few there are: the wavefronts that run ahead store a level's starts one after the
// other.  One level, with at most 128 / 256 / 512 / any number of spans: 1000 steps 16x16 binary 40.1 / 42.1 / 53.9 / 77.8, 64x64 dungeon
// 54.9 / 59.5 / 75.6 / 109, 4000 steps 115 / 108 / 111 / 286, 133 / 123 / 131 / 232; eight levels, 4000 steps 145 / 125 / 121 / 121.
constexpr int64_t kMostSpans = 256;
inline int64_t span_levels(int rows, int problem, bool observed, int64_t batch) {
  const bool binary = problem == PCGRL_BINARY;
  int64_t levels;
  if (rows == 16) levels = batch <= 128 ? 4096 : observed || batch <= 1024 ? 8192 : 16384;
  else if (rows == 32) levels = batch <= 512 || (observed && !binary) ? 4096 : observed || batch <= 2048 ? 8192 : 16384;
  else levels = batch <= 512 ? 2048 : observed ? 4096 : 8192;
  return std::min(levels, kMostSpans * batch);
}

// The most levels that any rollout of a context has side by side.
inline int64_t span_room(int rows, int problem, int64_t batch) {
  const int64_t most = std::max(span_levels(rows, problem, false, batch), span_levels(rows, problem, true, batch)) / batch * batch;
  return batch <= 4096 && most >= 2 * batch ? most : 0;
}

// It pays where the batch leaves the machine idle and the rollout is long enough for what the cutting costs:
// a second launch, 3 to 5 us in which one wavefront a level runs ahead, and the metrics from scratch.  How long that is depends on
// what a step costs otherwise, where a relay of 256 levels (a workgroup for each compute unit) is at its best.  Us as one / cut up,
// 9-cell windows (with 31 cells the same within a few percent):
//   16 rows  12 steps of 64 binary levels 15.0 / 12.4, maze 1.11 times as many a second, dungeon 1.02; of 256 dungeon levels (14) 1.08, (12) 0.98;
//            of 1024 binary levels 25.0 / 21.2, of 2048 27.9 / 28.6 (14 steps 1.02), of 3072 maze levels 25.7 / 26.9 (1.01)
//   32 rows  14 steps of 64 binary levels 1.21, maze 1.01, dungeon 1.00; 16 steps of 256 binary levels 1.18, maze 13.7 / 14.4, dungeon 15.0 / 16.5,
//            22 steps 1.00, 1.00; 512 maze levels, 22 steps 1.06; with 15 cells 2048 maze levels, 32 steps 45.2 / 48.1
//   64 rows  16 steps of 8 binary levels 1.19, maze 1.10, dungeon 1.00; 20 steps of 64 binary levels 1.08, maze 17.2 / 17.8 (25 steps 1.03),
//            dungeon 19.1 / 22.0 (30 steps 1.02); 256 binary levels, 32 steps 1.16, maze 1.00 (37 steps 1.02), dungeon 27.9 / 30.3 (48 steps 1.05);
//            1024 levels, 80 steps 1.21, 85 steps 1.08, 96 steps 1.08
// Beyond 256 levels, and with windows that a relay does not take, cutting pays from the start: 345 32x32 dungeon levels with 38 cells, 32 steps 56 / 33,
// 231 64x56 ones with 63 cells 46 / 42, 917 16x16 ones with 34 cells, 16 steps 38 / 29.
// (Smaller levels have less to find from scratch: 64 dungeon levels of 48x48, 20 steps 0.95, of 64x32 0.99, of 8x64 1.20; 256 of 32x17, 16 steps 0.99.)
// Without observations a rollout is one wavefront a level group, which is the longer chain: 64 16x16 maze levels, 200 steps
// 199 / 20 us, 4096 279 / 152, 2048 with 32 steps 44 / 27; 512 64x64 ones with 32 steps 47 / 28, 2048 57 / 57.
// Nor where the stores are what a rollout waits for: 1024 16x16 dungeon levels (7.9 MB a step) 53 / 43, 2048 maze levels
// (9.8 MB) 61 / 58, 1500 dungeon levels (11.5 MB) 75 / 80; 64x64 dungeon levels, 640 (4.9 MB) 1.08, 768 (5.9 MB) 0.94.  With wide windows and
// all compute units busy a relay stores 5.9 TB/s into a ring that spills from the cache and spans 4.8: 256 16x16 maze levels with 63 cells,
// 96 steps (490 MB) 85 / 104, 36 steps 1.05, but 320 of them 163 / 127; 448 of them (8.9 MB), 18 steps 27.3 / 30.9.
// And less where levels start again on the way, which is one more draw in a row for the wavefront that runs ahead and a longer chain for
// the span that has it: with a limit of 150 changes 64 64x64 dungeon levels, 30 steps 0.91, 45 steps 1.08, 256 32x32 ones, 22 steps 0.90, 33 steps
// 1.01, 64 16x16 ones, 12 steps 0.97; with 40 changes or 30 steps 768 64x64 dungeon levels 0.87 to 1.02 however long, 1024
// binary ones 0.92 to 1.27, 2048 levels without observations 0.91 to 1.02.  (A lane draws a row: 64 dungeon levels of 64x8, 20 steps 1.12, of 64x32 0.91.)
inline SpanShape span_shape(const SpanCase& c) {
  const SpanShape whole = {1, (int)c.steps};
  const int64_t B = c.batch, MB = (int64_t)1 << 20;
  const bool binary = c.problem == PCGRL_BINARY, dungeon = c.problem == PCGRL_DUNGEON;
  const bool restarts = c.episode > 0 && c.episode < 400, often = c.episode > 0 && c.episode < 60;
  const bool one_each = B <= 256;  // workgroups of a relay for a compute unit
  // the fewest steps; how many more where a relay is at its best; and twelfths of them more where levels start again
  int64_t most_batch = 4096, most_bytes = 9 * MB, fewest, more = 0, again = 0;
  if (!c.observed) {
    if (c.rows == 64 && often) most_batch = 1024;
    fewest = c.rows == 16 ? 8 + B / 128 : c.rows == 32 ? 8 + B / 96 : 12 + B / 32;
  } else if (c.rows == 16) {
    most_batch = 3072;
    fewest = 12;
    if (dungeon ? B > 64 && one_each : binary ? B > 1536 && B <= 2048 : B > 2048) more = 2;
    if (more > 0 || (dungeon && B <= 512)) again = 2;
  } else if (c.rows == 32) {
    most_batch = binary ? 3072 : 1536;
    fewest = 14 + B / 96;
    if (binary) {
      again = B > 1536 ? 4 : 0;
    } else {
      if (one_each && c.cells > 700) more = std::max<int64_t>(std::min<int64_t>(9 + B / 20, 22) - fewest, 0);
      again = one_each ? (dungeon ? (often ? 9 : 6) : 3) : B <= (dungeon ? 512 : 768) ? (often ? 5 : 2) : 0;
    }
  } else {
    const int64_t from32 = std::clamp<int64_t>(B - 32, 0, 32);
    if (one_each && !binary)
      more = (dungeon ? from32 / 4 + B / 32 : from32 / 8) * std::clamp<int64_t>(c.cells - 1536, 0, 2560) / 2560;
    fewest = 16 + B / 16;
    if (dungeon && B > 700) most_bytes = 5 * MB;
    if (dungeon && c.max_w > 16) again = one_each || often ? (B <= 384 ? 5 : 24) : B <= 384 ? 3 : 9;
    if (!dungeon && !binary && c.max_w > 32) again = one_each ? 3 : often ? 8 : 0;
    most_batch = !often ? 1024 : binary ? 900 : again == 0 ? 1024 : 640;
  }
  // (a wide window makes the steps themselves longer)
  const int64_t narrow = std::clamp<int64_t>(9500 - c.window_bits, 0, 1500);
  fewest += more * narrow / 1500;
  if (restarts) fewest += fewest * again * narrow / (12 * 1500);
  if (!binary && !dungeon && c.obs_bytes >= 8192) most_bytes = std::min(most_bytes, 8 * MB);
  if (B > most_batch || c.steps < fewest || c.step_bytes > most_bytes) return whole;
  const bool busy = 4 * B >= 3 * 256 * ((B + 255) / 256);
  if (c.obs_bytes >= (c.rows == 16 ? 16000 : 10000) && busy && c.step_bytes > (binary ? 8 * MB : 15 * MB / 4) && c.step_bytes * c.steps > 300 * MB)
    return whole;
  const int64_t spans = std::min(c.steps, span_levels(c.rows, c.problem, c.observed, B) / B);
  if (spans < 2) return whole;
  SpanShape s;
  s.steps = (int)((c.steps + spans - 1) / spans);
  s.spans = (int)((c.steps + s.steps - 1) / s.steps);
  return s;
}

}  // namespace pcgrl

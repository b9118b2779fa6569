// Whether, and into how many spans, a pcgrl_rollout is cut up along its steps.  Plain C++, apart from the
// kernels, so that the rule can be called on the host for batches and rollouts of any size.
#pragma once
#include <algorithm>
#include <cstdint>

namespace pcgrl {

struct SpanCase {
  int rows;                // of the size class
  bool binary;             // the binary problem
  bool observed;           // with observations, a slot for every step
  int64_t batch, steps;    // levels, steps of the rollout
  int64_t step_bytes;      // of the observations of a step
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
inline int64_t span_levels(int rows, bool binary, bool observed, int64_t batch) {
  if (rows == 16) return batch <= 128 ? 4096 : observed || batch <= 1024 ? 8192 : 16384;
  if (rows == 32) return batch <= 512 || (observed && !binary) ? 4096 : observed || batch <= 2048 ? 8192 : 16384;
  return batch <= 512 ? 2048 : observed ? 4096 : 8192;
}

// The most levels that any rollout of a context has side by side.
inline int64_t span_room(int rows, bool binary, int64_t batch) {
  const int64_t most = std::max(span_levels(rows, binary, false, batch), span_levels(rows, binary, true, batch)) / batch * batch;
  return batch <= 4096 && most >= 2 * batch ? most : 0;
}

// It pays where the batch leaves the machine idle and the rollout is long enough for what the cutting costs:
// a second launch, 3 to 5 us in which one wavefront a level runs ahead, and the metrics from scratch.  Us as one / cut up,
// 31-cell windows unless it says otherwise:
//   16 rows  64 binary levels, 4 steps 8.0 / 11.5, 8 steps 12.4 / 12.3, 12 steps 13.8 / 12.8, 16 steps 17.5 / 13.4, 256 steps 147 / 31;
//            64 maze levels, 12 steps 11.6 / 10.1; 1024 binary levels, 8 steps 20.8 / 19.4, 32 steps 53 / 33; 2048, 32 steps 62 / 47;
//            3000, 16 steps 51 / 42; with 9 cells 4096 binary levels, 32 steps 63 / 67, maze levels 49.8 / 49.3
//   32 rows  64 maze levels, 12 steps 11.7 / 12.3, 16 steps 13.8 / 12.6; 512 maze levels, 16 steps 18.7 / 19.2, 64 steps 47 / 34;
//            1024 maze levels, 32 steps 46 / 34; 2048 (15 cells) 45.2 / 48.1, binary ones 64 / 56; 3000 binary levels (9 cells) 87 / 68
//   64 rows  64 maze levels, 16 steps 16.4 / 15.1, 24 steps 20.9 / 16.3; 256 levels, 8 steps 13.6 / 17.3, 32 steps 26.9 / 26.4;
//            512 levels, 16 steps 22.1 / 26.2, 64 steps 55 / 49; 1024 levels, 32 steps 50 / 49, 128 steps (9 cells) 137 / 114
// Nor where the stores are what a rollout waits for: 1024 16x16 dungeon levels (7.9 MB a step) 53 / 43, 2048 maze levels
// (9.8 MB) 61 / 58, 1500 dungeon levels (11.5 MB) 75 / 80; with 63 cells 256 16x16 maze levels (5 MB) 34 / 31, 512 (10 MB) 119 / 125.
// Without observations a rollout is one wavefront a level group, which is the longer chain: 64 16x16 maze levels, 200 steps
// 199 / 20 us, 4096 279 / 152, 2048 with 32 steps 44 / 27; 512 64x64 ones with 32 steps 47 / 28, 2048 57 / 57.
inline SpanShape span_shape(const SpanCase& c) {
  const SpanShape whole = {1, (int)c.steps};
  const int64_t B = c.batch;
  int64_t most_batch, fewest;
  if (c.observed) {
    most_batch = c.rows == 16 ? 3072 : c.rows == 32 ? (c.binary ? 3072 : 1536) : 1024;
    fewest = c.rows == 16 ? 12 : c.rows == 32 ? 14 + B / 96 : 16 + B / 16;
  } else {
    most_batch = 4096;
    fewest = c.rows == 16 ? 8 + B / 128 : c.rows == 32 ? 8 + B / 96 : 12 + B / 32;
  }
  if (B > most_batch || c.steps < fewest || c.step_bytes > ((int64_t)9 << 20)) return whole;
  const int64_t spans = std::min(c.steps, span_levels(c.rows, c.binary, c.observed, B) / B);
  if (spans < 2) return whole;
  SpanShape s;
  s.steps = (int)((c.steps + spans - 1) / spans);
  s.spans = (int)((c.steps + s.steps - 1) / s.steps);
  return s;
}

}  // namespace pcgrl

// Which bytes of the plain layout a thread of get_state_kernel writes.  Plain C++, apart from the
// kernel, so that the arithmetic can be called on the host at sizes no test would allocate.
#pragma once
#include <cstdint>

namespace pcgrl {

constexpr int kGetThreads = 256;       // a workgroup of get_state_kernel
constexpr int kGetBytes = 16;          // consecutive cells a thread writes at a time
// A launch may have fewer than 2^32 threads in a direction, while 2^24 levels of 64 x 64 cells are 2^32
// pieces: beyond this many workgroups (2^30 threads, more than there can be levels) the launch gets rows
// of that many.
constexpr uint32_t kGetRow = 1u << 22;

struct GetGrid {
  uint32_t x, y;
};
// Workgroups for `batch` levels of `cells` cells: a thread for every piece of the cell arrays, if any
// is asked for, and at least one for every level's scalars.
constexpr GetGrid get_grid(uint32_t batch, uint32_t cells, bool with_cells) {
  const uint64_t pieces = with_cells ? ((uint64_t)batch * cells + kGetBytes - 1) / kGetBytes : 0;
  const uint64_t threads = pieces > batch ? pieces : batch;
  const uint64_t blocks = (threads + kGetThreads - 1) / kGetThreads;
  return {blocks < kGetRow ? (uint32_t)blocks : kGetRow, (uint32_t)((blocks + kGetRow - 1) / kGetRow)};
}

struct GetPiece {
  uint64_t at;       // the first of its cells, counted through the whole array
  int n;             // how many cells, 16 but for the last piece; none behind the end of the array
  int env, y, x;     // the level, row and column of the first one
};

// The piece of thread `thread` of workgroup (bx, by).
constexpr GetPiece get_piece(uint32_t bx, uint32_t by, int thread, uint32_t batch, int cells, int max_w) {
  const uint64_t total = (uint64_t)batch * (uint64_t)cells;
  const uint64_t first = ((uint64_t)by * kGetRow + bx) * (uint64_t)(kGetThreads * kGetBytes);
  GetPiece p = {first + (uint64_t)(kGetBytes * thread), 0, 0, 0, 0};
  if (p.at < total) {
    const int from = (int)(first % (uint32_t)cells) + kGetBytes * thread;  // (the 64-bit division is the whole workgroup's)
    p.n = total - p.at < (uint64_t)kGetBytes ? (int)(total - p.at) : kGetBytes;
    p.env = (int)(first / (uint32_t)cells) + from / cells;
    p.y = from % cells / max_w;
    p.x = from % cells % max_w;
  }
  return p;
}

// The level whose scalars a thread writes, if there is one of that number.
constexpr uint64_t get_level(uint32_t bx, uint32_t by, int thread) { return ((uint64_t)by * kGetRow + bx) * kGetThreads + (uint64_t)thread; }

}  // namespace pcgrl

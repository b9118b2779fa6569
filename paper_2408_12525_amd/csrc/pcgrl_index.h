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

// The sizes of the arrays, with what stands for a division by each on the device, where one takes some twenty
// vector instructions, and a 64-bit one hundreds: r, the largest 32-bit number over the divisor d.  The upper half of
// n r is the quotient or one less, as r d >= 2^32 - d, so that n r / 2^32 > n / d - 1 for every n < 2^32.
struct GetSizes {
  uint64_t total;                     // cells of all levels
  uint32_t cells, max_w;              // of a level, of its rows
  uint32_t per_level, per_row;        // see above
};
constexpr GetSizes get_sizes(uint32_t batch, int cells, int max_w) {
  return {(uint64_t)batch * (uint64_t)cells, (uint32_t)cells, (uint32_t)max_w, 0xffffffffu / (uint32_t)cells, 0xffffffffu / (uint32_t)max_w};
}
constexpr uint32_t divided(uint32_t n, uint32_t by, uint32_t reciprocal, uint32_t& rest) {
  const uint32_t q = (uint32_t)(((uint64_t)n * reciprocal) >> 32);
  rest = n - q * by;
  const bool more = rest >= by;
  rest -= more ? by : 0u;
  return q + (more ? 1u : 0u);
}

// The piece of thread `thread` of workgroup (bx, by).
constexpr GetPiece get_piece(uint32_t bx, uint32_t by, int thread, const GetSizes& s) {
  const uint64_t first = ((uint64_t)by * kGetRow + bx) * (uint64_t)(kGetThreads * kGetBytes);
  GetPiece p = {first + (uint64_t)(kGetBytes * thread), 0, 0, 0, 0};
  if (p.at < s.total) {
    uint32_t level = 0, rest = 0, x = 0;  // (the first cell's: the whole workgroup's)
    if (s.total <= 0xffffffffu) {
      level = divided((uint32_t)first, s.cells, s.per_level, rest);
    } else {
      level = (uint32_t)(first / s.cells);
      rest = (uint32_t)(first % s.cells);
    }
    p.n = s.total - p.at < (uint64_t)kGetBytes ? (int)(s.total - p.at) : kGetBytes;
    p.env = (int)(level + divided(rest + (uint32_t)(kGetBytes * thread), s.cells, s.per_level, rest));
    p.y = (int)divided(rest, s.max_w, s.per_row, x);
    p.x = (int)x;
  }
  return p;
}
constexpr GetPiece get_piece(uint32_t bx, uint32_t by, int thread, uint32_t batch, int cells, int max_w) {
  return get_piece(bx, by, thread, get_sizes(batch, cells, max_w));
}

// The level whose scalars a thread writes, if there is one of that number.
constexpr uint64_t get_level(uint32_t bx, uint32_t by, int thread) { return ((uint64_t)by * kGetRow + bx) * kGetThreads + (uint64_t)thread; }

}  // namespace pcgrl

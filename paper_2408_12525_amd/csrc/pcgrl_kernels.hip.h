// Device code of the batched PCGRL step for gfx950 (wave64).
//
// Layout.  A level lives in registers as row bitboards: lane (g, y) of a wavefront holds row y of
// the level in group g, one word per tile-code bit-plane (bit x = column x).  S = 16, 32 or 64 is
// the padded side; a wavefront therefore carries G = 64 / S levels.  Vertical neighbours are
// reached with DPP lane shifts, horizontal ones with word shifts, so one breadth-first layer of a
// whole level is a handful of full-rate vector instructions and no memory traffic.  LDS is used
// only to stage the observation as a packed bit stream before it is widened to bytes.
//
// Everything a group shares (shape, position, metrics, ...) is held redundantly in every lane of
// the group; "uniform" below means uniform inside one group.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "pcgrl_index.h"
#include "pcgrl_relay.h"
#include "pcgrl_split.h"

namespace pcgrl {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
// The same in the global address space: stores through a plain pointer whose origin the compiler
// has lost sight of become flat instructions, which also count against the LDS counter.
typedef __attribute__((address_space(1))) u32x4 global_u32x4;
typedef __attribute__((address_space(1))) uint8_t global_u8;

constexpr int kMaxMetrics = 16;
// the largest bit-packed observation: 63 x 63 cells, seven tile types, border and pinpoint channel
constexpr int kMaxPackedRow = (63 * 63 * 9 + 7) / 8;

enum : int { kBinary = 0, kMaze = 1, kDungeon = 2 };
enum : int { kPadBorder = 0, kPadWall = 1 };
enum : int { kPosScan = 0, kPosRandom = 1 };
enum : int { kRegionsIncremental = 0, kRegionsRecount = 1 };
// step kernel variants: one step per launch; the same with the work of a wavefront split over a metrics
// wavefront and observation wavefronts of one workgroup; n steps per launch; n steps per launch split the
// same way; that with observation wavefronts that take the steps in turn; and that for one span of a rollout,
// from the state its levels have there (see span_starts_kernel).  (A relay, see rollout_relay_kernel, is a
// kernel of its own.)
enum : int { kModeStep = 0, kModeSplit = 1, kModeRollout = 2, kModeRolloutSplit = 3, kModeRolloutTurns = 4, kModeSpan = 5 };

// Per-environment scalars, 32 bytes, read and written as two 16-byte words.
struct __attribute__((aligned(16))) EnvRec {
  uint8_t h, w, py, px;
  int32_t t;
  int32_t n_changes;
  int32_t episode;
  uint64_t key;          // generator key of (seed, env, episode)
  uint32_t cell_frozen;  // the agent's current cell is a pinpoint
  uint32_t pad_;
};
static_assert(sizeof(EnvRec) == 32, "EnvRec must be 32 bytes");

struct KArgs {
  // the first 64 bytes are everything a step needs to request its loads: one scalar fetch
  void* planes;      // word [P][plane_stride], index env * S + y
  void* frozen;      // word [plane_stride]
  EnvRec* env;       // [B_pad]
  int32_t* metrics;  // [B_pad][16]
  uint32_t* targets; // [B_pad][16], lo | hi << 16 (ranges are clamped to 0..65535); the 16 words in front of it: the reward weights (float)
  const int32_t* actions;
  int32_t B, plane_stride;
  int32_t envs_per_wave_log2;  // bits 0-7: log2 of the distinct levels per wavefront (at most 64 / S);
                               // bits 8-15, split step only: the same for an observation wavefront;
                               // bits 16-23, split rollout only: log2 of the observation wavefronts
                               // that take the steps in turn; bits 24-30: of the searching wavefronts
  int32_t use_frozen;     // 0: no level of this context has a pinpoint cell; bit 1: a step needs the pinpoint rows (they are shown in the observation)
  uint8_t* obs;
  float* reward;
  uint8_t* done;
  unsigned long long* bad_actions;
  uint64_t seed;
  int32_t max_h, max_w, min_h, min_w;
  int32_t obs_w, pad_mode, pos_mode, n_frozen, max_steps, max_changes, autoreset, regions_mode;
  int32_t env_obs_bytes;  // bytes from one level's observation to the next: C * obs_w * obs_w, or an eighth (rounded up) when packed, or the configured pitch
  int32_t obs_packed;     // non-zero: bit-packed observation format
  int32_t obs_frozen_channel;  // non-zero: a last channel marks the pinpoint cells in view
  int32_t stream_obs;     // how observations are stored: kStoreCached / kStoreStream / kStoreThrough
  int32_t by_die;       // rollouts: consecutive level groups run on the same die (see level_group_of_block)
  int32_t fresh;          // init kernel only: first levels from the seed instead of the stored ones
  int32_t rollout_steps;  // rollout kernel: steps per launch
  int32_t obs_slots;      // rollout kernel: step t writes observation slot t % obs_slots
  int32_t obs_lds_words;  // split step: LDS words of one observation wavefront's staging area
  uint32_t cdf[8];
  int32_t target_lo[kMaxMetrics], target_hi[kMaxMetrics];
  int32_t pinpoint_tile[8];
  uint32_t ctrl_mask;
  int32_t ctrl_lo[kMaxMetrics], ctrl_hi[kMaxMetrics];
};

// The step kernel's argument block read
// through a pointer the optimiser cannot trace back to the arguments.  Blocks that run once in
// thousands of steps (a level restarting) read their configuration through it: loads made this way
// stay inside the block, whereas loads from the by-value argument are hoisted, with all the scalar
// arithmetic that depends on them, to the top of the kernel where every wavefront pays for them.
// fill_rest_of_args() below reads the whole block this way at a point of the caller's choosing.
// (In the single-step kernel the block comes after the arguments that are handed over in
// registers, in the rollout kernel it is the only argument: ROLL says which kernel is running.)
constexpr int kStepArgsOffset = 56;
template <bool ROLL> __device__ __forceinline__ const KArgs& cold_args() {
  auto seg = __builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(seg));
  return *(const KArgs*)((const char*)seg + (ROLL ? 0 : kStepArgsOffset));
}

// Completes an argument block of which only the fields that came in registers are set (`hot`:
// the six state pointers, B, plane_stride, envs_per_wave_log2, use_frozen) with everything else
// from the block in memory.  The fetch, and the wait for it, stay where this is called.
__device__ __forceinline__ void fill_rest_of_args(KArgs& hot) {
  KArgs t = cold_args<false>();
  t.planes = hot.planes;
  t.frozen = hot.frozen;
  t.env = hot.env;
  t.metrics = hot.metrics;
  t.targets = hot.targets;
  t.actions = hot.actions;
  t.B = hot.B;
  t.plane_stride = hot.plane_stride;
  t.envs_per_wave_log2 = hot.envs_per_wave_log2;
  t.use_frozen = hot.use_frozen;
  hot = t;
}

template <int S> struct RowWord { using T = uint32_t; };
template <> struct RowWord<64> { using T = uint64_t; };

template <int PROBLEM> struct Prob;
template <> struct Prob<kBinary> { static constexpr int K = 2, P = 1, M = 4, CNT = 2; };
template <> struct Prob<kMaze> { static constexpr int K = 4, P = 2, M = 6, CNT = 2; };
template <> struct Prob<kDungeon> { static constexpr int K = 7, P = 3, M = 10, CNT = 3; };

// --------------------------------------------------------------- generator
// Counter-based numbers: the mixing function of the published splitmix64 generator applied to
// key + golden * (stream, counter).  Integer only, so CPU and GPU agree bit for bit.

__device__ __forceinline__ uint64_t mix64(uint64_t z) {
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}
constexpr uint64_t kGolden = 0x9E3779B97F4A7C15ull;
__device__ __forceinline__ uint64_t env_key(uint64_t seed, uint64_t env, uint64_t episode) {
  uint64_t k0 = mix64(seed + kGolden * (env + 1));
  return mix64(k0 ^ (0xD1B54A32D192ED03ull * (episode + 1)));
}
__device__ __forceinline__ uint64_t draw(uint64_t key, uint32_t stream, uint32_t counter) {
  uint64_t c = ((uint64_t)stream << 32) + (uint64_t)counter + 1;
  return mix64(key + kGolden * c);
}
__device__ __forceinline__ int below(uint32_t r, int n) { return (int)__umulhi(r, (uint32_t)n); }

// ------------------------------------------------------------ lane algebra

template <int CTRL> __device__ __forceinline__ uint32_t dpp_zero_fill(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xf, 0xf, true);
}
constexpr int kRowShr1 = 0x111, kRowShl1 = 0x101, kWaveShr1 = 0x138, kWaveShl1 = 0x130;

// Flood layers written out.  A lane-shifted (DPP) read has to come two instructions after the write of
// any register the instruction uses, and the compiler neither looks into an assembly block for that
// nor lets anything read a block's result without a wait; so whole groups of layers are one block, in
// an order that leaves few waits.  Measured, clocks a layer of one wavefront alone: 32 / 43 for 16 / 32
// rows (41 / 65 layer by layer as the compiler arranges it), 54 / 78 for two sets together.  Each is the
// variant with the fewest vector instructions; one more per set and no waits at all was slower where
// the batch fills the machine (32x32 binary levels at 16 384: 13.9 against 13.5 us per step).  Every
// lane shift rides on a two-operand OR.  bitop3:0xa8 is (first | second) & third.
#define PCGRL_DPP(D, F, ACC, SHIFT, ROWS) "v_or_b32_dpp " D ", " F ", " ACC " " SHIFT ":1 row_mask:" ROWS " bank_mask:0xf bound_ctrl:1\n\t"
// one layer of the set F inside R, to D; scratch %2, %3
#define PCGRL_LAYER16(F, D, R)                                             \
  "v_lshrrev_b32 %2, 1, " F "\n\tv_lshl_or_b32 %2, " F ", 1, %2\n\t"       \
  PCGRL_DPP("%3", F, F, "row_shr", "0xf") "s_nop 0\n\t"                    \
  PCGRL_DPP("%2", F, "%2", "row_shl", "0xf")                               \
  "v_bitop3_b32 " D ", %2, %3, " R " bitop3:0xa8\n\t"
// (32 rows: a shift inside each row of 16 lanes, then the step across the middle of each level only:
// rows 1 and 3 take from below them, rows 0 and 2 from above them; what the second step repeats does
// no harm)
#define PCGRL_LAYER32(F, D, R)                                             \
  "v_lshrrev_b32 %2, 1, " F "\n\tv_lshl_or_b32 %2, " F ", 1, %2\n\t"       \
  PCGRL_DPP("%3", F, F, "row_shr", "0xf") "s_nop 0\n\t"                    \
  PCGRL_DPP("%2", F, "%2", "row_shl", "0xf")                               \
  PCGRL_DPP("%3", F, "%3", "wave_shr", "0xa") "s_nop 0\n\t"                \
  PCGRL_DPP("%2", F, "%2", "wave_shl", "0x5")                              \
  "v_bitop3_b32 " D ", %2, %3, " R " bitop3:0xa8\n\t"
// one layer of king's moves of two sets, %2 and %3, inside %8, to DA and DB; scratch %4 to %7
#define PCGRL_KINGS16(DA, DB)                                                               \
  PCGRL_DPP("%4", "%2", "%2", "row_shr", "0xf") "s_nop 0\n\t"                               \
  PCGRL_DPP("%6", "%3", "%3", "row_shr", "0xf") PCGRL_DPP("%4", "%2", "%4", "row_shl", "0xf") \
  "v_lshrrev_b32 %5, 1, %4\n\t"                                                             \
  PCGRL_DPP("%6", "%3", "%6", "row_shl", "0xf")                                             \
  "v_lshl_or_b32 %5, %4, 1, %5\n\tv_bitop3_b32 " DA ", %5, %4, %8 bitop3:0xa8\n\t"          \
  "v_lshrrev_b32 %7, 1, %6\n\tv_lshl_or_b32 %7, %6, 1, %7\n\t"                              \
  "v_bitop3_b32 " DB ", %7, %6, %8 bitop3:0xa8\n\t"
#define PCGRL_KINGS32(DA, DB)                                                               \
  PCGRL_DPP("%4", "%2", "%2", "row_shr", "0xf") "s_nop 0\n\t"                               \
  PCGRL_DPP("%6", "%3", "%3", "row_shr", "0xf") PCGRL_DPP("%4", "%2", "%4", "row_shl", "0xf") \
  "s_nop 0\n\t"                                                                             \
  PCGRL_DPP("%6", "%3", "%6", "row_shl", "0xf") PCGRL_DPP("%4", "%2", "%4", "wave_shr", "0xa") \
  "s_nop 0\n\t"                                                                             \
  PCGRL_DPP("%6", "%3", "%6", "wave_shr", "0xa") PCGRL_DPP("%4", "%2", "%4", "wave_shl", "0x5") \
  "v_lshrrev_b32 %5, 1, %4\n\t"                                                             \
  PCGRL_DPP("%6", "%3", "%6", "wave_shl", "0x5")                                            \
  "v_lshl_or_b32 %5, %4, 1, %5\n\tv_bitop3_b32 " DA ", %5, %4, %8 bitop3:0xa8\n\t"          \
  "v_lshrrev_b32 %7, 1, %6\n\tv_lshl_or_b32 %7, %6, 1, %7\n\t"                              \
  "v_bitop3_b32 " DB ", %7, %6, %8 bitop3:0xa8\n\t"

template <int S> struct Lanes {
  using W = typename RowWord<S>::T;
  static constexpr int G = 64 / S;
  int lane, g, y, gbase;
  __device__ __forceinline__ Lanes() {
    lane = (int)(threadIdx.x & 63u);
    g = lane / S;
    y = lane % S;
    gbase = g * S;
  }
  // value held by the lane of row y-1 of the same level (0 for the top row)
  __device__ __forceinline__ W from_above(W v) const {
    if constexpr (S == 16) {
      return dpp_zero_fill<kRowShr1>(v);
    } else if constexpr (S == 32) {
      uint32_t r = dpp_zero_fill<kWaveShr1>(v);
      return y == 0 ? 0u : r;
    } else {
      uint32_t lo = dpp_zero_fill<kWaveShr1>((uint32_t)v);
      uint32_t hi = dpp_zero_fill<kWaveShr1>((uint32_t)(v >> 32));
      return ((uint64_t)hi << 32) | lo;
    }
  }
  // value held by the lane of row y+1 (0 for the bottom row)
  __device__ __forceinline__ W from_below(W v) const {
    if constexpr (S == 16) {
      return dpp_zero_fill<kRowShl1>(v);
    } else if constexpr (S == 32) {
      uint32_t r = dpp_zero_fill<kWaveShl1>(v);
      return y == S - 1 ? 0u : r;
    } else {
      uint32_t lo = dpp_zero_fill<kWaveShl1>((uint32_t)v);
      uint32_t hi = dpp_zero_fill<kWaveShl1>((uint32_t)(v >> 32));
      return ((uint64_t)hi << 32) | lo;
    }
  }
  // the same for a 32-bit value of any size class
  __device__ __forceinline__ uint32_t from_above32(uint32_t v) const {
    const uint32_t r = S == 16 ? dpp_zero_fill<kRowShr1>(v) : dpp_zero_fill<kWaveShr1>(v);
    return S == 32 && y == 0 ? 0u : r;
  }
  __device__ __forceinline__ uint32_t from_below32(uint32_t v) const {
    const uint32_t r = S == 16 ? dpp_zero_fill<kRowShl1>(v) : dpp_zero_fill<kWaveShl1>(v);
    return S == 32 && y == S - 1 ? 0u : r;
  }
  // acc | the value of `v` a lane shift away, as one instruction.  (The compiler folds a lane shift
  // into an OR that is the only use of it, but would first gather a chain of ORs into three-operand
  // ones, which cannot take a shifted operand; the empty statement keeps the chain as it is written.)
  template <int CTRL, int ROWS = 0xf> static __device__ __forceinline__ uint32_t or_shifted(uint32_t acc, uint32_t v) {
    uint32_t r = acc | (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xf, ROWS == 0xf);
    asm("" : "+v"(r));
    return r;
  }
  // a cell set with the cells above and below it
  __device__ __forceinline__ W with_above_below(W f) const {
    if constexpr (S == 16) {
      return or_shifted<kRowShl1>(or_shifted<kRowShr1>(f, f), f);
    } else if constexpr (S == 32) {
      // a shift inside each row of 16 lanes, then the step across the boundary between the two
      // rows of one level only (rows 1 and 3 take from below them, rows 0 and 2 from above them);
      // the second step repeats values the first has already ORed in, which does no harm
      const uint32_t u = or_shifted<kWaveShr1, 0xa>(or_shifted<kRowShr1>(f, f), f);
      return or_shifted<kWaveShl1, 0x5>(or_shifted<kRowShl1>(u, f), f);
    } else {
      const uint32_t lo = (uint32_t)f, hi = (uint32_t)(f >> 32);
      return ((uint64_t)or_shifted<kWaveShl1>(or_shifted<kWaveShr1>(hi, hi), hi) << 32) |
             or_shifted<kWaveShl1>(or_shifted<kWaveShr1>(lo, lo), lo);
    }
  }
  // one breadth-first layer inside the cell set r
  __device__ __forceinline__ W grow(W f, W r) const { return dilate(f) & r; }
  // the four-neighbour dilation of a cell set (the set itself included), not masked
  __device__ __forceinline__ W dilate(W f) const { return with_above_below(f) | (W)(f << 1) | (W)(f >> 1); }
  // one layer of king's moves inside the cell set r
  __device__ __forceinline__ W grow8(W f, W r) const {
    const W v = with_above_below(f);
    return (v | (W)(v << 1) | (W)(v >> 1)) & r;
  }
  // Two breadth-first layers: `one` after the first, the result after the second.
  __device__ __forceinline__ W grow_twice(W f, W r, W& one) const {
    if constexpr (S == 64) {
      one = grow(f, r);
      return grow(one, r);
    } else {
      uint32_t two, t, u;
      if constexpr (S == 16)
        asm(PCGRL_LAYER16("%4", "%0", "%5") PCGRL_LAYER16("%0", "%1", "%5")
            : "=&v"(one), "=&v"(two), "=&v"(t), "=&v"(u) : "v"(f), "v"(r));
      else
        asm(PCGRL_LAYER32("%4", "%0", "%5") PCGRL_LAYER32("%0", "%1", "%5")
            : "=&v"(one), "=&v"(two), "=&v"(t), "=&v"(u) : "v"(f), "v"(r));
      return two;
    }
  }
  // N layers of king's moves of two sets side by side; a1 and b1 are what they were one layer earlier.
  template <int N> __device__ __forceinline__ void grow8_both(W& a, W& b, W& a1, W& b1, W r) const {
    static_assert(N == 2 || N == 4, "written out for two and for four layers");
    a1 = a;
    b1 = b;
    if constexpr (S == 64) {
#pragma unroll
      for (int l = 0; l < N - 1; ++l) {
        a1 = grow8(a1, r);
        b1 = grow8(b1, r);
      }
      a = grow8(a1, r);
      b = grow8(b1, r);
    } else {
      uint32_t u, v, x, y;
#define PCGRL_OPERANDS : "=&v"(a), "=&v"(b), "+&v"(a1), "+&v"(b1), "=&v"(u), "=&v"(v), "=&v"(x), "=&v"(y) : "v"(r)
      if constexpr (S == 16 && N == 2)
        asm("s_nop 1\n\t" PCGRL_KINGS16("%2", "%3") PCGRL_KINGS16("%0", "%1") PCGRL_OPERANDS);
      else if constexpr (S == 16)
        asm("s_nop 1\n\t" PCGRL_KINGS16("%2", "%3") PCGRL_KINGS16("%2", "%3") PCGRL_KINGS16("%2", "%3")
            PCGRL_KINGS16("%0", "%1") PCGRL_OPERANDS);
      else if constexpr (N == 2)
        asm("s_nop 1\n\t" PCGRL_KINGS32("%2", "%3") PCGRL_KINGS32("%0", "%1") PCGRL_OPERANDS);
      else
        asm("s_nop 1\n\t" PCGRL_KINGS32("%2", "%3") PCGRL_KINGS32("%2", "%3") PCGRL_KINGS32("%2", "%3")
            PCGRL_KINGS32("%0", "%1") PCGRL_OPERANDS);
#undef PCGRL_OPERANDS
    }
  }
  // bits of a wave ballot that belong to this lane's group, moved down to bit 0
  __device__ __forceinline__ uint64_t gbits(uint64_t ballot) const {
    if constexpr (S == 64) return ballot;
    return (ballot >> gbase) & ((1ull << S) - 1ull);
  }
  __device__ __forceinline__ bool gany(bool pred) const {
    return gbits(__builtin_amdgcn_ballot_w64(pred)) != 0;
  }
  // rotate by N lanes inside each row of 16 lanes / exchange with the lane 16 away
  template <int N> static __device__ __forceinline__ int ror(int v) {
    return __builtin_amdgcn_update_dpp(v, v, 0x120 + N, 0xf, 0xf, false);
  }
  static __device__ __forceinline__ int xor16(int v) { return __builtin_amdgcn_ds_swizzle(v, 0x401F); }
  // sum / maximum over the lanes of the group, returned in every lane
  __device__ __forceinline__ int gsum(int v) const {
    v += ror<8>(v);
    v += ror<4>(v);
    v += ror<2>(v);
    v += ror<1>(v);
    if constexpr (S >= 32) v += xor16(v);
    if constexpr (S == 64) v = __builtin_amdgcn_readlane(v, 0) + __builtin_amdgcn_readlane(v, 32);
    return v;
  }
  __device__ __forceinline__ int gmax(int v) const {
    v = max(v, ror<8>(v));
    v = max(v, ror<4>(v));
    v = max(v, ror<2>(v));
    v = max(v, ror<1>(v));
    if constexpr (S >= 32) v = max(v, xor16(v));
    if constexpr (S == 64) v = max(__builtin_amdgcn_readlane(v, 0), __builtin_amdgcn_readlane(v, 32));
    return v;
  }
  // value of lane `row` of this group
  __device__ __forceinline__ W gread(W v, int row) const { return (W)__shfl(v, gbase + row); }
  __device__ __forceinline__ int gread_i(int v, int row) const { return __shfl(v, gbase + row); }
};

__device__ __forceinline__ int popc(uint32_t v) { return __popc(v); }
__device__ __forceinline__ int popc(uint64_t v) { return __popcll(v); }
__device__ __forceinline__ int ctz(uint32_t v) { return __ffs(v) - 1; }
__device__ __forceinline__ int ctz(uint64_t v) { return __ffsll((unsigned long long)v) - 1; }

template <int S> __device__ __forceinline__ bool wave_any(bool pred) {
  return __builtin_amdgcn_ballot_w64(pred) != 0;
}

// The cell with the lowest row-major index of a set, as a one-cell set (empty if the set is).
template <int S>
__device__ __forceinline__ typename RowWord<S>::T first_cell(const Lanes<S>& L,
                                                             typename RowWord<S>::T set) {
  using W = typename RowWord<S>::T;
  uint64_t rows = L.gbits(__builtin_amdgcn_ballot_w64(set != 0));
  int first_row = rows ? ctz(rows) : -1;
  return L.y == first_row ? (W)(set & (~set + 1)) : (W)0;
}

// ---------------------------------------------------------------- tile planes

template <int PROBLEM, typename W>
__device__ __forceinline__ W channel_row(const W (&p)[Prob<PROBLEM>::P], W inside, int c) {
  W r = inside;
#pragma unroll
  for (int i = 0; i < Prob<PROBLEM>::P; ++i) r &= ((c >> i) & 1) ? p[i] : (W)~p[i];
  return r;
}

// ------------------------------------------------------------------ metrics
// Floods test for their end after every second layer at first and, after this many such trips,
// after every fourth layer: most floods are over within a few layers, but the test and the jump
// back cost about as much as three layers, which long floods need not pay every time.
constexpr int kShortTrips = 2;

// Floods all levels of a wavefront of several until none grows any more, keeping of each what its last layers
// are worked out from afterwards: the cells at the end of its last trip that still grew (`base`), those one
// layer before (`before`), and how many layers that is.  Kept once a trip and for the level as a whole, where a lane
// for itself would have to be looked at after every second layer: for 32-row levels, whose floods are long.  Us without / with:
// steps of 4096 32x32 binary levels with 15 cells 8.99 / 8.84, of 8192 10.9 / 10.3, 16 384 13.1 / 12.6, 32 768 18.6 / 18.1, of 16 384 levels of random
// shapes from 8x8 on 13.0 / 12.8; 512 levels cut into spans, 32 steps 36.7 / 35.0; 1024 exact diameters 27.6 / 26.3, but 4096 59.5 / 59.8, 16 384
// 160.6 / 163.3; levels installed or reset the same.  16-row levels, four to a wavefront, are faster where a batch is small (8192 with 15 cells 6.9 /
// 6.7) and slower where it is large (65 536 19.1 / 19.7), and their rollouts would lose a wavefront a SIMD to the registers.  Nor for
// rollouts of large batches (65 536 32x32 levels 19.5 / 19.7 us a step).
template <int S>
__device__ __forceinline__ int flood_to_end(const Lanes<S>& L, typename RowWord<S>::T seed, typename RowWord<S>::T pass,
                                            typename RowWord<S>::T& base, typename RowWord<S>::T& before) {
  using W = typename RowWord<S>::T;
  W V = seed;
  int k = 0;
  base = seed;
  before = 0;
  auto trip = [&](auto n_tag) {
    constexpr int N = decltype(n_tag)::value;
    W one = V, two = V;
#pragma unroll
    for (int l = 0; l < N; l += 2) two = L.grow_twice(two, pass, one);
    const uint64_t grew = __builtin_amdgcn_ballot_w64(two != one);
    const bool mine = L.gbits(grew) != 0;
    base = mine ? two : base;
    before = mine ? one : before;
    k += mine ? N : 0;
    V = two;
    return grew != 0;
  };
  bool more = true;
  for (int n = 0; n < kShortTrips && more; ++n) more = trip(std::integral_constant<int, 2>{});
  while (more) more = trip(std::integral_constant<int, 4>{});
  return k;
}

// One sweep of the two-sweep diameter estimate: breadth-first layers from `seed` inside `pass`.
// Returns the eccentricity of the seed and leaves in `last` the cells of the last layer
// (the seed itself when nothing else is reachable) and in `comp` all the cells reached.  The loop advances two layers per trip and
// only remembers, per lane, what the last pair of layers that reached the lane added; which of the
// two layers was the last one is worked out after the loop with one more layer from the cells
// known before that pair.
template <int S, bool TRIPS = S == 32>
__device__ __forceinline__ int sweep(const Lanes<S>& L, typename RowWord<S>::T seed,
                                     typename RowWord<S>::T pass, typename RowWord<S>::T& last,
                                     typename RowWord<S>::T& comp) {
  using W = typename RowWord<S>::T;
  if constexpr (TRIPS) {  // (see flood_to_end)
    W base, before, one;
    const int k = flood_to_end<S>(L, seed, pass, base, before);
    const W two = L.grow_twice(base, pass, one), three = L.grow(two, pass);
    const W l3 = three & ~two, l2 = two & ~one, l1 = one & ~base;
    const bool a3 = L.gany(l3 != 0), a2 = L.gany(l2 != 0), a1 = L.gany(l1 != 0);
    last = a3 ? l3 : a2 ? l2 : a1 ? l1 : (W)(base & ~before);
    comp = three;
    return k + (a3 ? 3 : a2 ? 2 : a1 ? 1 : 0);
  }
  W V = seed, added = seed;
  int k = 0, k_last = 0;  // pairs done; the pair that last added cells in this lane
  auto pair_of_layers = [&]() {
    W V1;
    const W V2 = L.grow_twice(V, pass, V1);
    k += 1;
    if (V2 != V) {
      added = V2 ^ V;
      k_last = k;
    }
    V = V2;
    return V2 != V1;  // a second layer that adds nothing means the flood is complete
  };
  bool more = true;
  for (int n = 0; n < kShortTrips && more; ++n) more = wave_any<S>(pair_of_layers());
  while (more) {  // (long floods test for the end every fourth layer only, as the region search does)
    pair_of_layers();
    more = wave_any<S>(pair_of_layers());
  }
  const int kk = L.gmax(k_last);               // the last pair that added cells to the level
  const W pair = k_last == kk ? added : (W)0;  // what it added
  const W before = V & ~pair;
  const W first = L.grow(before, pass) & ~before;
  const W second = pair & ~first;
  const bool two = L.gany(second != 0);
  last = two ? second : first;
  comp = V;  // every cell the sweep reached: the component of the seed
  return kk == 0 ? 0 : 2 * kk - (two ? 0 : 1);
}

// The eccentricity alone.
template <int S, bool TRIPS = S == 32>
__device__ __forceinline__ int eccentricity(const Lanes<S>& L, typename RowWord<S>::T seed,
                                            typename RowWord<S>::T pass) {
  using W = typename RowWord<S>::T;
  if constexpr (TRIPS) {  // (see flood_to_end)
    W base, before, one;
    const int k = flood_to_end<S>(L, seed, pass, base, before);
    const W two = L.grow_twice(base, pass, one), three = L.grow(two, pass);
    return k + (L.gany(three != two) ? 3 : L.gany(two != one) ? 2 : L.gany(one != base) ? 1 : 0);
  }
  W V = seed;
  int k = 0, k1 = 0, k2 = 0;  // pairs done; the pairs whose first / second layer last reached this lane
  auto pair_of_layers = [&]() {
    W V1;
    const W V2 = L.grow_twice(V, pass, V1);
    k += 1;
    if (V1 != V) k1 = k;
    const bool grew = V2 != V1;
    if (grew) k2 = k;
    V = V2;
    return grew;
  };
  bool more = true;
  for (int n = 0; n < kShortTrips && more; ++n) more = wave_any<S>(pair_of_layers());
  while (more) {
    pair_of_layers();
    more = wave_any<S>(pair_of_layers());
  }
  return L.gmax(max(2 * k2, 2 * k1 - 1));
}

// Binary domain, footnote: sweep from the first walkable cell x, then from the far end of the
// longest shortest path out of x (lowest row-major index among equally far cells).
// `comp` receives the component of x: the estimate depends on nothing else (see
// diameter_untouched).
template <int S, bool TRIPS = S == 32>
__device__ __forceinline__ int two_sweep_diameter(const Lanes<S>& L, typename RowWord<S>::T pass,
                                                  typename RowWord<S>::T& comp) {
  using W = typename RowWord<S>::T;
  W x = first_cell<S>(L, pass);
  W far;
  sweep<S, TRIPS>(L, x, pass, far, comp);
  W y = first_cell<S>(L, far);
  return eccentricity<S, TRIPS>(L, y, pass);
}

// Whether an edit leaves the two-sweep estimate as it is.  The estimate is a function of x, the
// first walkable cell, and of the component of x alone (both sweeps stay inside it, and the far
// end is chosen among its cells).  An edit that flips the walkability of a cell which neither
// lies in that component nor touches it leaves the component as it is; x stays the first walkable
// cell unless the edited cell became walkable and comes before it in row-major order (an x that
// is walled up lies in the component).  `comp` is the component of x before the edit (empty if no
// cell was walkable), `cell` the edited cell as a one-cell set in its row's lane, `dcell` its
// dilation; (py, px) its coordinates.
template <int S>
__device__ __forceinline__ bool diameter_untouched(const Lanes<S>& L, typename RowWord<S>::T comp,
                                                   typename RowWord<S>::T cell, typename RowWord<S>::T dcell,
                                                   int py, int px, bool now_walkable) {
  const bool touched = L.gany((dcell & comp) != 0);
  const uint64_t rows = L.gbits(__builtin_amdgcn_ballot_w64(comp != 0));
  const int xrow = rows ? ctz(rows) : S;  // row of x (none: every cell comes before it)
  const bool before = L.gany(cell != 0 && (py < xrow || (py == xrow && px < ctz(comp))));
  return !touched && !(now_walkable && before);
}

// Distance from a source set to the nearest cell of a target set, -1 if none is reachable.
// `reached` receives the target cells found in the layer of the first hit.  A trip looks for the
// target in its last layer only; which layer of the trip met it first is worked out when that
// happens, from the layers the trip has kept.
template <int S>
__device__ __forceinline__ int nearest(const Lanes<S>& L, typename RowWord<S>::T src,
                                       typename RowWord<S>::T tgt, typename RowWord<S>::T pass,
                                       typename RowWord<S>::T& reached) {
  using W = typename RowWord<S>::T;
  W V = src;
  int d = -1, it = 0;
  reached = 0;
  auto trip = [&](auto n_tag) {
    constexpr int N = decltype(n_tag)::value;
    W layer[N];
#pragma unroll
    for (int l = 0; l < N; l += 2) layer[l + 1] = L.grow_twice(l == 0 ? V : layer[l - 1], pass, layer[l]);
    const bool ch = layer[N - 1] != layer[N - 2];
    V = layer[N - 1];
    const bool hit = d < 0 && L.gany((V & tgt) != 0);
    if (wave_any<S>(hit)) {
      int first = N - 1;
#pragma unroll
      for (int l = N - 2; l >= 0; --l)
        if (L.gany((layer[l] & tgt) != 0)) first = l;
      if (hit) {
        d = it + first + 1;
        W at = layer[N - 1];
#pragma unroll
        for (int l = N - 2; l >= 0; --l) at = first == l ? layer[l] : at;
        reached = at & tgt;
      }
    }  // (the level's flood may go on while others search: nothing reads it any more)
    it += N;
    return wave_any<S>(ch && d < 0);  // a last layer that adds nothing means the flood is complete
  };
  bool more = true;
  for (int n = 0; n < kShortTrips && more; ++n) more = trip(std::integral_constant<int, 2>{});
  while (more) more = trip(std::integral_constant<int, 4>{});
  return d;
}

// Dungeon: one flood from the players that looks for keys and enemies at the same time.
template <int S>
__device__ __forceinline__ void nearest_two(const Lanes<S>& L, typename RowWord<S>::T src,
                                            typename RowWord<S>::T tgt_a, typename RowWord<S>::T tgt_b,
                                            typename RowWord<S>::T pass, int& d_a,
                                            typename RowWord<S>::T& reached_a, int& d_b) {
  using W = typename RowWord<S>::T;
  W V = src;
  int it = 0;
  d_a = -1;
  d_b = -1;
  reached_a = 0;
  auto trip = [&](auto n_tag) {
    constexpr int N = decltype(n_tag)::value;
    W layer[N];
#pragma unroll
    for (int l = 0; l < N; l += 2) layer[l + 1] = L.grow_twice(l == 0 ? V : layer[l - 1], pass, layer[l]);
    const bool ch = layer[N - 1] != layer[N - 2];
    V = layer[N - 1];
    const bool hit_a = d_a < 0 && L.gany((V & tgt_a) != 0);
    const bool hit_b = d_b < 0 && L.gany((V & tgt_b) != 0);
    if (wave_any<S>(hit_a || hit_b)) {
      int first_a = N - 1, first_b = N - 1;
#pragma unroll
      for (int l = N - 2; l >= 0; --l) {
        if (L.gany((layer[l] & tgt_a) != 0)) first_a = l;
        if (L.gany((layer[l] & tgt_b) != 0)) first_b = l;
      }
      if (hit_a) {
        d_a = it + first_a + 1;
        W at = layer[N - 1];
#pragma unroll
        for (int l = N - 2; l >= 0; --l) at = first_a == l ? layer[l] : at;
        reached_a = at & tgt_a;
      }
      if (hit_b) d_b = it + first_b + 1;
    }
    it += N;
    const bool finished = d_a >= 0 && d_b >= 0;
    return wave_any<S>(ch && !finished);
  };
  bool more = true;
  for (int n = 0; n < kShortTrips && more; ++n) more = trip(std::integral_constant<int, 2>{});
  while (more) more = trip(std::integral_constant<int, 4>{});
}

// The cells of a level that lie on its border (next to nothing on some side).
template <int S>
__device__ __forceinline__ typename RowWord<S>::T border_cells(const Lanes<S>& L, typename RowWord<S>::T inside) {
  using W = typename RowWord<S>::T;
  return inside & ~(L.from_above(inside) & L.from_below(inside) & (W)(inside << 1) & (W)(inside >> 1));
}

// Number of 4-connected components of `pass`, the walkable cells of a level.
//
// In the plane it is the Euler number - cells less neighbouring pairs plus 2 x 2 squares, which every
// lane counts for its row - plus the number of holes, i.e. of components of the walls, diagonal steps
// included, that do not reach the outside.  A flood of king's moves from the border through the walls
// leaves the walls of the holes; those are counted by parallel shrinking (Levialdi's algorithm): in one
// step, on every cell at once, a cell stays if its left, lower or lower-left neighbour is set, and an
// empty cell is filled if its left and its lower neighbour are; this moves every component towards the
// lower left corner of its bounding box without joining two or splitting one, until it is a single
// cell with no neighbour, which the next step deletes: the count is the number of such cells met on
// the way.  Holes are few and small where the walkable region itself, shrunk the same way (in the
// 4-connected form: a cell stays if its left or its lower neighbour is set, an empty one is filled if
// left, lower and lower-left all are), takes up to h + w - 1 steps: on generated 64x64 levels with 45 %
// walls 43 layers of 10 vector instructions and 11 steps of 23 against 67 steps of 20, with 25 % 13 and
// 22 against 126.  Shrinking the walkable cells remains for levels of mostly walls (`open` false), whose
// components are small, and for those whose walls wind so much that the flood takes more than 2 S
// layers; it needs no more than 2 S steps whatever the level looks like.  8192 generated 64x64 maze levels,
// reset with observations: 59.0 -> 47.6 us against shrinking the walkable cells throughout.
template <int S>
__device__ __forceinline__ int regions_full(const Lanes<S>& L, typename RowWord<S>::T pass, typename RowWord<S>::T inside,
                                            bool open) {
  using W = typename RowWord<S>::T;
  if (wave_any<S>(open)) {
    const W walls = inside & ~pass;
    W out = walls & border_cells<S>(L, inside);
    bool more = true;
    for (int trip = 0; trip < S / 2 && more; ++trip) {
      W before = out;
#pragma unroll
      for (int n = 0; n < 3; ++n) before = L.grow8(before, walls);
      out = L.grow8(before, walls);
      more = wave_any<S>(out != before);
    }
    if (!more) {
      const W down = pass & L.from_above(pass);
      int count = popc(pass) - popc((W)(pass & (W)(pass >> 1))) - popc(down) + popc((W)(down & (W)(down >> 1)));
      W p = walls & ~out;
      while (wave_any<S>(p != 0)) {  // (at most 2 S steps)
#pragma unroll
        for (int n = 0; n < 2; ++n) {
          const W left = (W)(p << 1), below = L.from_below(p);
          const W beside = left | (W)(p >> 1), three = beside | p;
          count += popc((W)(p & ~(beside | L.from_above(three) | L.from_below(three))));
          p = (p & (left | below | (W)(below << 1))) | (left & below);
        }
      }
      return L.gsum(count);
    }
  }
  W p = pass;
  int vanished = 0;  // this row's share of the count
  for (int trip = 0; trip < S / 2 && wave_any<S>(p != 0); ++trip) {  // (2 S steps: more than any level needs)
#pragma unroll
    for (int n = 0; n < 4; ++n) {
      const W left = (W)(p << 1), below = L.from_below(p);
      const W keep = p & (left | below);
      vanished += popc((W)(p & ~(keep | (W)(p >> 1) | L.from_above(p))));
      p = keep | (below & (W)((W)(p & below) << 1));
    }
  }
  return L.gsum(vanished);
}

// How many components of a level without the cell (py, px) touch that cell, i.e. by how much more or
// less than one the region count changes when the cell's walkability does.  `pass` holds the walkable
// cells without it, `cell` the cell itself in its row's lane (nothing of either in a level that does
// not ask: the answer is then 0).
//
// The eight cells around it, taken as a ring, answer at once where their walkable cells form a single
// arc (an arc counts if it holds one of the four neighbours; an open corner between two walls does
// not and is taken as a wall).  With n arcs, n > 1, there are n arcs of walls between them, and in the
// plane the two tell about each other: two arcs of walkable cells hang together outside the ring
// exactly if no wall path, diagonal steps included, joins the walls on either side of them.  So the
// number of components among the arcs is n + 1 less the number of wall components among the wall arcs,
// where everything outside the map is one wall.  The walls are what is searched: their steps are
// king's moves and the way round the outside is free, so that the search is short where one among the
// walkable cells winds about (64x64 maze in mid-episode, layers of a search at the 99th percentile: 28
// against 47 with two floods among the walkable cells and 150 with one).  Two floods go on side by
// side, from one wall arc and from all the others, until they meet or either stalls.
template <int S>
__device__ __forceinline__ int components_around(const Lanes<S>& L, typename RowWord<S>::T pass, typename RowWord<S>::T inside,
                                                 typename RowWord<S>::T cell, int h, int w, int py, int px) {
  using W = typename RowWord<S>::T;
  const uint32_t row = (uint32_t)(px > 0 ? pass >> (px - 1) : (W)(pass << 1)) & 7u;  // left, middle, right
  // ring, clockwise from the upper left cell (bit 0), in the lane of the cell
  const uint32_t lower = L.from_below32(row);
  uint32_t open = L.from_above32(row) | ((row & 4u) << 1) | ((row & 1u) << 7) | (__brev(lower) >> 25);
  const uint32_t twice = open | (open << 8);
  open &= 0xaau | (twice >> 7) | (twice >> 1);
  open = cell != 0 ? open : 0u;
  uint32_t wall_starts = ~open & ((open | (open << 8)) >> 7) & 0xffu;  // one cell of every wall arc
  wall_starts = cell != 0 ? wall_starts : 0u;
  const int packed = (int)(wall_starts | (open << 8));
  const uint32_t all = (uint32_t)(S == 64 ? __builtin_amdgcn_readlane(packed, __builtin_amdgcn_readfirstlane(py)) : L.gread_i(packed, py));
  const int arcs = popc(all & 0xffu);
  bool go = arcs > 1;
  int k = arcs > 0 ? arcs : all != 0 ? 1 : 0;
  if (wave_any<S>(go)) {
    const uint32_t mid = ((wall_starts >> 7) & 1u) | ((wall_starts >> 1) & 4u);
    const uint32_t seed = mid | L.from_below32(wall_starts & 7u) | L.from_above32((__brev(wall_starts) >> 25) & 7u);
    const W walls = go ? inside & ~(pass | cell) : (W)0;
    W U = (px > 0 ? (W)seed << (px - 1) : (W)(seed >> 1)) & walls;
    const W edge = walls & border_cells<S>(L, inside);
    // wall arcs still to be taken: those of which U holds a cell, and all that lie outside as one
    const uint32_t off_map = (py == 0 ? 0x07u : 0u) | (py == h - 1 ? 0x70u : 0u) | (px == 0 ? 0xc1u : 0u) | (px == w - 1 ? 0x1cu : 0u);
    bool out = go && (all & off_map & 0xffu) != 0;
    int left = go ? popc(all & ~off_map & 0xffu) + (out ? 1 : 0) : 0;
    while (wave_any<S>(left >= 2)) {
      W A = out ? edge : first_cell<S>(L, U);
      if (!out) U &= ~A;
      out = false;
      W B = U;
      if (left < 2) A = B = 0;
      bool meet;
      auto trip = [&](auto n_tag) {
        constexpr int N = decltype(n_tag)::value;
        W A1, B1;
        L.template grow8_both<N>(A, B, A1, B1, walls);
        if (L.gany((A & edge) != 0)) A |= edge;
        if (L.gany((B & edge) != 0)) B |= edge;
        const bool grew_a = L.gany(A != A1), grew_b = L.gany(B != B1);
        meet = L.gany((A & B) != 0);
        return wave_any<S>(grew_a & grew_b & !meet);
      };
      bool more = true;
      for (int n = 0; n < kShortTrips && more; ++n) more = trip(std::integral_constant<int, 2>{});
      while (more) more = trip(std::integral_constant<int, 4>{});
      if (left >= 2) {
        k -= meet ? 0 : 1;
        left -= 1;
      }
    }
  }
  return k;
}

// The same number searched for among the walkable cells: of distinct components of `passw` (the level with
// the edited cell walled off) among the walkable neighbours `nbr` of that cell.  A flood starts from the
// first neighbour; if it has not reached the others within a few layers, a second one starts from those
// and the two go on side by side until they meet or either stalls.  For binary levels of 16 rows, and of 32
// in rollouts, whose components are small: with two or four of them to a wavefront, what the ring costs every
// edit is more than the searches through their walls save (262 144 16x16 levels, steps without observations
// 34.8 against 37.3 us, 256-step rollouts of 64 of them 152 against 155; 65 536 32x32 levels with a 3-cell
// window, rollouts 19.8 against 20.3 us a step, 16 384 of them 6.26 against 6.45).  A single step of 32-row levels
// lasts as long as its slowest search, which is shorter through the walls, and other problems are faster so
// as well (16x16 dungeons at 65 536 18.4 against 18.8, at 4096 4.58 against 4.73).
template <int S>
__device__ __forceinline__ int neighbour_components(const Lanes<S>& L, typename RowWord<S>::T nbr,
                                                    typename RowWord<S>::T passw) {
  using W = typename RowWord<S>::T;
  W U = nbr;
  // at most four cells in three rows; a row holds two of them only for the left/right pair
  auto count = [&](W u) {
    int rows = popc(L.gbits(__builtin_amdgcn_ballot_w64(u != 0)));
    return rows + (L.gany((u & (u - 1)) != 0) ? 1 : 0);
  };
  int left = count(U);
  int k = 0;
  for (;;) {
    bool go = left >= 2;
    if (!go && left == 1) {
      k += 1;
      left = 0;
      U = 0;
    }
    if (!wave_any<S>(go)) break;
    W A = go ? first_cell<S>(L, U) : (W)0;
    W pw = go ? passw : (W)0;
    // A group whose neighbours are all reached is finished for good: whatever its flood still
    // adds while other groups go on changes nothing below.
    bool more = true;
    for (int n = 0; n < kShortTrips && more; ++n) {
      W A1;
      const W An = L.grow_twice(A, pw, A1);
      bool ch = An != A1;  // a last layer that adds nothing means the flood is complete
      A = An;
      bool open = L.gany((U & ~A) != 0);
      more = wave_any<S>(ch && open);
    }
    U &= ~A;
    bool meet = false;
    if (more) {
      W B = U;
      do {
        W A1, B1;
        A = L.grow_twice(L.grow_twice(A, pw, A1), pw, A1);
        B = L.grow_twice(L.grow_twice(B, pw, B1), pw, B1);
        const bool grew_a = L.gany(A != A1), grew_b = L.gany(B != B1);
        meet = L.gany((A & B) != 0);
        more = wave_any<S>(grew_a & grew_b & !meet);
      } while (more);
    }
    k += go && !meet ? 1 : 0;
    left = count(U);
  }
  return k;
}

// Full metric vector of the level held by a group (all M entries).
template <int S, int PROBLEM, bool TRIPS = S == 32>
__device__ __forceinline__ void full_metrics(const Lanes<S>& L,
                                             const typename RowWord<S>::T (&p)[Prob<PROBLEM>::P],
                                             typename RowWord<S>::T inside, bool active,
                                             int (&m)[Prob<PROBLEM>::M], typename RowWord<S>::T& comp) {
  using W = typename RowWord<S>::T;
  using PR = Prob<PROBLEM>;
  comp = 0;  // binary problem: the component of the first walkable cell (kept with the level)
  W in = active ? inside : (W)0;
  W wall = channel_row<PROBLEM, W>(p, in, 1);
  W pass = in & ~wall;
#pragma unroll
  for (int k = 0; k < PR::K; ++k) m[PR::CNT + k] = L.gsum(popc(channel_row<PROBLEM, W>(p, in, k)));
  int cells = 0;
#pragma unroll
  for (int k = 0; k < PR::K; ++k) cells += m[PR::CNT + k];
  m[0] = regions_full<S>(L, pass, in, 5 * m[PR::CNT + 1] <= 3 * cells);
  if constexpr (PROBLEM == kBinary) {
    m[1] = two_sweep_diameter<S, TRIPS>(L, pass, comp);
  } else if constexpr (PROBLEM == kMaze) {
    W r;
    int d = nearest<S>(L, channel_row<PROBLEM, W>(p, in, 2), channel_row<PROBLEM, W>(p, in, 3), pass, r);
    m[1] = d < 0 ? 0 : d;
  } else {
    W k1, r;
    int d1, de;
    nearest_two<S>(L, channel_row<PROBLEM, W>(p, in, 2), channel_row<PROBLEM, W>(p, in, 3),
                   channel_row<PROBLEM, W>(p, in, 5), pass, d1, k1, de);
    int d2 = nearest<S>(L, k1, channel_row<PROBLEM, W>(p, in, 4), pass, r);
    m[1] = (d1 >= 0 && d2 >= 0) ? d1 + d2 : 0;
    m[2] = de < 0 ? 0 : de;
  }
}

__device__ __forceinline__ int loss(int v, int lo, int hi) { return max(0, max(lo - v, v - hi)); }
// a target range as it is kept on the device
__device__ __forceinline__ uint32_t pack_range(int lo, int hi) {
  return (uint32_t)min(max(lo, 0), 65535) | ((uint32_t)min(max(hi, 0), 65535) << 16);
}

// Target of a controlled metric for the episode with generator key `key` (Methods / Training).
__device__ __forceinline__ uint32_t control_target(const KArgs& a, uint64_t key, int i) {
  int v = a.ctrl_lo[i] + below((uint32_t)(draw(key, 4, (uint32_t)i) >> 32), a.ctrl_hi[i] - a.ctrl_lo[i] + 1);
  return pack_range(v, v);
}

template <typename W> __device__ __forceinline__ W inside_row(int y, int h, int w) {
  W full = w >= (int)(8 * sizeof(W)) ? (W)~(W)0 : (W)(((W)1 << w) - 1);
  return y < h ? full : (W)0;
}

// ---------------------------------------------------------------- episodes

// Cells drawn side by side by a level that restarts inside a step or a rollout.  What a draw waits for
// counts where a launch lasts as long as its slowest wavefront (steps of 4096 64x64 maze levels with a change limit,
// four / two / one: 12.9 / 13.6 / 13.9 us), registers and length of code where none restarts: 8192 64x64
// maze levels 11.92 / 11.63 / 11.64 us a step, 16 384 16x16 dungeon levels 8.61 / 8.43 / 8.46 (with a limit 10.93 /
// 10.91 / 10.95), and 97 instead of 96 vector registers for 32x32 dungeons with wide windows (17 000 levels with 33
// cells 27.4 us with four, 25.6 with two).  In a rollout wavefronts are not in step, and the constants of several
// hashes are scalar registers that its loop lacks (8192 64x64 dungeon levels 6.9 / 6.6 / 6.6 us a step).
template <int S, int PROBLEM, bool ROLL>
constexpr int kDrawsAbreast = ROLL ? 1 : PROBLEM == kDungeon || (S == 64 && PROBLEM == kMaze) ? 2 : 4;

// Start of an episode: shape, tiles, pinpoints, first position, all from the env's key.  SHARED: inside a
// step, where few levels of a wavefront begin one.  ABREAST: how many cells are drawn side by side.
template <int S, int PROBLEM, bool SHARED = false, int ABREAST = 4>
__device__ __forceinline__ void begin_episode(const KArgs& a, const Lanes<S>& L, uint64_t key,
                                              typename RowWord<S>::T (&p)[Prob<PROBLEM>::P],
                                              typename RowWord<S>::T& fz, int& h, int& w, int& py,
                                              int& px, bool restart = true, int envl = 0) {
  using W = typename RowWord<S>::T;
  using PR = Prob<PROBLEM>;
  h = a.max_h;
  w = a.max_w;
  if (a.min_h < a.max_h) h = a.min_h + below((uint32_t)(draw(key, 0, 0) >> 32), a.max_h - a.min_h + 1);
  if (a.min_w < a.max_w) w = a.min_w + below((uint32_t)(draw(key, 0, 1) >> 32), a.max_w - a.min_w + 1);
  bool empty_start = true;
#pragma unroll
  for (int k = 0; k < 8; ++k) empty_start = empty_start && a.cdf[k] == 0;
#pragma unroll
  for (int i = 0; i < PR::P; ++i) p[i] = 0;
  // Bits x0 .. x0 + n - 1 of this row (n <= 32 and the same in all lanes), as they would be in a level
  // of any size.  Bound by vector instructions, six of the 22 or so a cell being 32-bit multiplications
  // of the hash.  The rest is kept short: the counter goes down by one constant, so that a cell's bits
  // are shifted into 32-bit words from the right, as the carry of an addition, and end up in place,
  // and the thresholds, which are non-decreasing, are searched instead of counted (8192 64x64 maze levels,
  // reset with observations: 65.1 -> 57.1 us when this loop was brought in, 47.6 -> 46.3 with the carries).
  // The thresholds are fetched once and chosen among as values.  A choice between two of them written on
  // the argument block, or on an array, is a choice between two addresses: inside a step, where the block
  // is read through a pointer, each was a vector load per cell, two in a row for a draw, and each waited
  // for every observation store the wavefront still had under way.  Steps with a change limit of 100, us:
  // 8192 16x16 dungeon levels 13.1 -> 10.9, 4096 32x32 ones with three pinpoints 13.6 -> 10.8, 8192 64x64
  // ones 27.8 -> 22.7, 8192 16x16 maze levels 8.5 -> 7.7.
  uint32_t cdf[PR::K - 1];
#pragma unroll
  for (int i = 0; i < PR::K - 1; ++i) {
    cdf[i] = a.cdf[i];
    // (scalar registers are what the loops around a restart are short of; one threshold is no burden)
    if constexpr (PROBLEM != kBinary) asm("" : "+v"(cdf[i]));
  }
  auto either = [](bool c, uint32_t x, uint32_t y) { return c ? x : y; };
  auto draw_cells = [&](uint64_t k, int x0, int n, uint32_t (&acc)[PR::P]) {
#pragma unroll
    for (int i = 0; i < PR::P; ++i) acc[i] = 0;
    uint64_t z = k + kGolden * ((1ull << 32) + (uint64_t)(uint32_t)(L.y * a.max_w + x0 + n));
    auto cell = [&](uint64_t zc) {
      const uint32_t r = (uint32_t)(mix64(zc) >> 32);
      // acc = 2 acc + bit, the bits of a cell in one block: as the carry of an addition a bit takes one
      // instruction (a select and a shift otherwise); a comparison's result may be read two instructions
      // after it, which the compiler does not see to inside the block
      auto bits = [](bool c) { return __builtin_amdgcn_ballot_w64(c); };
      uint64_t none;
      if constexpr (PROBLEM == kBinary) {
        asm("s_nop 1\n\tv_addc_co_u32_e64 %0, %1, %0, %0, %2" : "+v"(acc[0]), "=&s"(none) : "s"(bits(r >= cdf[0])));
      } else if constexpr (PROBLEM == kMaze) {
        const bool b1 = r >= cdf[1];
        asm("s_nop 1\n\tv_addc_co_u32_e64 %0, %2, %0, %0, %3\n\tv_addc_co_u32_e64 %1, %2, %1, %1, %4"
            : "+v"(acc[0]), "+v"(acc[1]), "=&s"(none) : "s"(bits(r >= either(b1, cdf[2], cdf[0]))), "s"(bits(b1)));
      } else {  // (tile 7 does not exist)
        const bool b2 = r >= cdf[3];
        const bool b1 = r >= either(b2, cdf[5], cdf[1]);
        const bool b0 = r >= either(b1, cdf[2], either(b2, cdf[4], cdf[0]));
        asm("s_nop 1\n\tv_addc_co_u32_e64 %0, %3, %0, %0, %4\n\tv_addc_co_u32_e64 %1, %3, %1, %1, %5\n\t"
            "v_addc_co_u32_e64 %2, %3, %2, %2, %6"
            : "+v"(acc[0]), "+v"(acc[1]), "+v"(acc[2]), "=&s"(none)
            : "s"(bits(b0) & ~(bits(b1) & bits(b2))), "s"(bits(b1)), "s"(bits(b2)));
      }
    };
    int j = n;
    if constexpr (ABREAST > 1) {
      for (; j >= ABREAST; j -= ABREAST, z -= ABREAST * kGolden) {
#pragma unroll
        for (int i = 0; i < ABREAST; ++i) cell(z - i * kGolden);
      }
    }
#pragma unroll 1
    for (; j > 0; --j, z -= kGolden) cell(z);
  };
  if constexpr (SHARED && (64 / S) > 1) {
    // Inside a step few levels of a wavefront restart at the same time, and the draws are what a
    // restart costs: every lane group takes a G-th of the columns of a restarting level, whichever
    // group holds it, and the rows are put together across the groups afterwards.  Levels that
    // restart together take turns; copies of one level are served by the same turn.
    constexpr int G = 64 / S;
    uint64_t todo = empty_start ? 0ull : __builtin_amdgcn_ballot_w64(restart);
    while (todo != 0) {
      const int src = (int)__builtin_ctzll(todo);  // a lane of the first level still to do
      const uint64_t k = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(key >> 32), src) << 32) |
                         (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)key, src);
      const int kw = __builtin_amdgcn_readlane(w, src), kenv = __builtin_amdgcn_readlane(envl, src);
      const int n = (kw + G - 1) / G;
      uint32_t part[PR::P];
      draw_cells(k, L.g * n, n, part);
      const bool mine = restart && envl == kenv;
#pragma unroll
      for (int i = 0; i < PR::P; ++i) {
        uint32_t v = part[i] << (L.g * n);
        if constexpr (S == 16) v |= (uint32_t)Lanes<S>::xor16((int)v);
        v |= (uint32_t)__shfl_xor((int)v, 32);
        if (mine) p[i] = (W)v;
      }
      todo &= ~__builtin_amdgcn_ballot_w64(mine);
    }
  } else if (!empty_start) {
    int widest = __builtin_amdgcn_readfirstlane(w);
#pragma unroll
    for (int g = 1; g < 64 / S; ++g) widest = max(widest, __builtin_amdgcn_readlane(w, g * S));
#pragma unroll
    for (int x0 = 0; x0 < S; x0 += 32) {
      const int n = min(widest - x0, 32);
      if (n <= 0) break;
      uint32_t acc[PR::P];
      draw_cells(key, x0, n, acc);
#pragma unroll
      for (int i = 0; i < PR::P; ++i) p[i] |= (W)acc[i] << x0;
    }
  }
  {
    const W in = inside_row<W>(L.y, h, w);
#pragma unroll
    for (int i = 0; i < PR::P; ++i) p[i] &= in;
  }
  fz = 0;
  int placed = 0;
  for (uint32_t att = 0; att < 64 && placed < a.n_frozen; ++att) {
    uint64_t u = draw(key, 2, att);
    int fy = below((uint32_t)(u >> 32), h), fx = below((uint32_t)u, w);
    bool mine = L.y == fy;
    bool fresh = L.gany(mine && ((fz >> fx) & 1) == 0);
    if (fresh) {
      int ptile = -1;  // Task / Pinpoint tiles: a pivotal tile frozen at this cell
#pragma unroll
      for (int j = 0; j < 8; ++j) ptile = placed == j ? a.pinpoint_tile[j] : ptile;
      if (mine) {
        fz |= (W)1 << fx;
        if (ptile >= 0) {
#pragma unroll
          for (int i = 0; i < PR::P; ++i) p[i] = (p[i] & ~((W)1 << fx)) | ((W)((ptile >> i) & 1) << fx);
        }
      }
      ++placed;
    }
  }
  py = 0;
  px = 0;
  if (a.pos_mode == kPosRandom) {
    uint64_t u = draw(key, 3, 0);
    py = below((uint32_t)(u >> 32), h);
    px = below((uint32_t)u, w);
  }
}

// -------------------------------------------------------------- observation

// Orders this wavefront's LDS accesses (other lanes' writes before this lane's reads).  LDS
// operations of one wavefront execute in issue order, so only the compiler has to be told; the
// fence names the LDS address space so that no wait on global memory is generated.
__device__ __forceinline__ void lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
  __builtin_amdgcn_wave_barrier();
}

// How the lane groups of a wavefront are used.  A wavefront has G = 64 / S groups; `epw` of them
// carry distinct levels (slots), the remaining groups hold copies of those levels (copy > 0).
// Copies repeat the metric work for free (their lanes would idle otherwise) and share out the
// observation channels; only copy 0 stores results.  Small batches use fewer levels per wavefront
// so that more wavefronts, and with them more latency hiding, are in flight.
struct Slot {
  int slot, copy, copies, copies_log2;
};

// Where and how a wavefront writes its observations, as far as that does not depend on the levels
// themselves.  The window rows are first packed as a bit stream in LDS (bit j of the stream = byte j
// of the wavefront's contiguous output region, shifted so that 16-bit chunks line up with 16-byte
// aligned addresses), then every lane widens 16 bits to 16 bytes and issues one aligned 16-byte
// store.  A single-step kernel works the plan out, and clears the LDS words, while its loads are
// still in flight.
struct ObsPlan {
  uint8_t* base;     // 16-byte aligned address at or just below the wavefront's output region
  int dbytes, d;     // the region starts dbytes bytes = d stream bits after base
  int E, total;      // stream bits of one level, and of the wavefront (d included)
  int lane_off;      // stream position of this lane's level and first channel
  int q_lo, q_hi;    // aligned 16-byte chunks [q_lo, q_hi) lie wholly inside the region
  int edge_pos;      // the byte of the partial head (lanes 0-15) or tail (16-31) chunk this lane writes,
  bool edge_want;    // if any
  bool active;       // this lane group has a level
};

__device__ __forceinline__ ObsPlan obs_plan(const KArgs& a, int lane, const Slot& sl, uint8_t* obs,
                                            int env0, int nvalid) {
  ObsPlan pl;
  // One level's part of the stream is E bits long; its output is E bytes (one byte per bit) or,
  // bit-packed, E / 8 bytes.
  const bool packed = a.obs_packed != 0;
  pl.E = packed ? a.env_obs_bytes * 8 : a.env_obs_bytes;
  uint8_t* region = obs + (size_t)env0 * (size_t)a.env_obs_bytes;
  // The usual case -- the array and the distance between two levels' observations are multiples
  // of 16 bytes -- needs none of the edge arithmetic below (it runs on the scalar unit, which
  // all the wavefronts of a compute unit share: thirty instructions fewer per wavefront).
  if ((((uintptr_t)obs | (uintptr_t)(uint32_t)a.env_obs_bytes) & 15u) == 0) {
    pl.dbytes = 0;
    pl.base = region;
    pl.d = 0;
    pl.total = nvalid * pl.E;
    pl.lane_off = sl.slot * pl.E + sl.copy * (a.obs_w * a.obs_w);
    pl.active = sl.slot < nvalid;
    pl.q_lo = 0;
    pl.q_hi = (packed ? pl.total >> 3 : pl.total) >> 4;
    pl.edge_pos = 0;
    pl.edge_want = false;
    return pl;
  }
  pl.dbytes = (int)((uintptr_t)region & 15u);
  pl.base = region - pl.dbytes;
  pl.d = packed ? pl.dbytes * 8 : pl.dbytes;
  pl.total = pl.d + nvalid * pl.E;
  pl.lane_off = pl.d + sl.slot * pl.E + sl.copy * (a.obs_w * a.obs_w);
  pl.active = sl.slot < nvalid;
  // in bytes of output the region is [lo, hi) after base
  const int lo = pl.dbytes, hi = packed ? pl.total >> 3 : pl.total;
  pl.q_lo = (lo + 15) >> 4;
  pl.q_hi = hi >> 4;
  const int t = lane & 15;
  const bool is_tail = lane >= 16;
  const int q = is_tail ? pl.q_hi : 0;
  pl.edge_pos = (q << 4) + t;
  pl.edge_want = lane < 32 && (is_tail ? ((hi & 15) != 0 && (pl.q_hi > 0 || lo == 0)) : lo > 0) &&
                 pl.edge_pos >= lo && pl.edge_pos < hi;
  return pl;
}
// Keeps the plan's values where they were computed (the optimiser would otherwise move them next
// to their uses, behind the wait for the loads).
__device__ __forceinline__ void obs_plan_pin(ObsPlan& pl) {
  int ew = pl.edge_want ? 1 : 0, ac = pl.active ? 1 : 0;
  // (wave-uniform values all of them; said explicitly, since a value that merges two branches may
  // otherwise be given a vector register, which the constraints below cannot take)
  {
    const uintptr_t b = (uintptr_t)pl.base;
    pl.base = (uint8_t*)(((uintptr_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(b >> 32)) << 32) |
                         (uintptr_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)b));
    pl.dbytes = __builtin_amdgcn_readfirstlane(pl.dbytes);
    pl.d = __builtin_amdgcn_readfirstlane(pl.d);
    pl.E = __builtin_amdgcn_readfirstlane(pl.E);
    pl.total = __builtin_amdgcn_readfirstlane(pl.total);
    pl.q_lo = __builtin_amdgcn_readfirstlane(pl.q_lo);
    pl.q_hi = __builtin_amdgcn_readfirstlane(pl.q_hi);
  }
  asm volatile("" : "+s"(pl.base), "+s"(pl.dbytes), "+s"(pl.d), "+s"(pl.E), "+s"(pl.total), "+s"(pl.q_lo),
               "+s"(pl.q_hi), "+v"(pl.lane_off), "+v"(pl.edge_pos), "+v"(ew), "+v"(ac));
  pl.edge_want = ew != 0;
  pl.active = ac != 0;
}
// (16 bytes per lane and instruction: a wavefront's staging area is 16-byte aligned and a whole
// number of 16-byte pieces long, see the library's sizing of it)
__device__ __forceinline__ void obs_clear(uint32_t* lds, int lane, const ObsPlan& pl) {
  const int npieces = (pl.total + 127) >> 7;
  uint4* l4 = reinterpret_cast<uint4*>(__builtin_assume_aligned(lds, 16));
  for (int i = lane; i < npieces; i += 64) l4[i] = make_uint4(0u, 0u, 0u, 0u);
}

// Writes the observations of this wavefront's levels.  WIDE = window wider than 32; CLEARED = the
// LDS words of the stream are zero already; LEAN = the caller is a wavefront that does nothing but
// observations and can afford a copy of the channel code for every number of copies.
template <int S, int PROBLEM, bool WIDE, bool CLEARED, bool LEAN>
__device__ __forceinline__ void write_obs(const KArgs& a, const Lanes<S>& L, const Slot& sl,
                                          const ObsPlan& pl, uint32_t* lds,
                                          const typename RowWord<S>::T (&p)[Prob<PROBLEM>::P],
                                          typename RowWord<S>::T fz, typename RowWord<S>::T inside,
                                          int qy, int qx) {
  using W = typename RowWord<S>::T;
  using PR = Prob<PROBLEM>;
  using BW = typename std::conditional<WIDE, uint64_t, uint32_t>::type;  // one window row
  const int ow = a.obs_w, r = ow >> 1;
  const int Cfz = PR::K + (a.pad_mode == kPadBorder ? 1 : 0);  // index of the pinpoint channel, if any
  const int C = Cfz + (a.obs_frozen_channel ? 1 : 0);
  if constexpr (!CLEARED) obs_clear(lds, L.lane, pl);
  lds_sync();

  if (pl.active) {
    const BW owmask = WIDE ? (BW)((1ull << ow) - 1ull) : (BW)(0xffffffffu >> (32 - ow));
    const int y0 = qy - r, x0 = qx - r;
    const int sr = x0 > 0 ? x0 : 0, sl_ = x0 < 0 ? -x0 : 0;  // one of the two shifts is zero
    auto window = [&](W row) -> BW {
      if constexpr (WIDE || S == 64) return (BW)(((uint64_t)row >> sr) << sl_) & owmask;
      else return (BW)((row >> sr) << sl_) & owmask;
    };
    // the lane's own row seen through the window: each code plane and the inside mask
    BW wp[PR::P];
#pragma unroll
    for (int k = 0; k < PR::P; ++k) wp[k] = window(p[k]);
    const BW win_in = window(inside);
    const BW win_fz = window(fz) & win_in;
    const BW out_win = (BW)~win_in & owmask;  // window cells outside the map's columns
    const int padc = a.pad_mode == kPadBorder ? PR::K : 1;
    const int cstride = ow * ow;
    auto emit = [&](int off, BW bits) {  // ORs a window row into the stream at bit `off`
      const int w0 = off >> 5, sh = off & 31;
      if constexpr (WIDE) {
        uint64_t lo = bits << sh;
        uint32_t hi = sh ? (uint32_t)(bits >> (64 - sh)) : 0u;
        atomicOr(&lds[w0], (uint32_t)lo);
        atomicOr(&lds[w0 + 1], (uint32_t)(lo >> 32));
        if (hi) atomicOr(&lds[w0 + 2], hi);
      } else {
        // (both words unconditionally: a test for an empty upper half costs every lane a compare
        // and the wavefront two scalar instructions, an OR of zero costs nothing that matters; the
        // staging area has spare words behind the stream for the one that may fall past its end)
        uint64_t t = (uint64_t)bits << sh;
        atomicOr(&lds[w0], (uint32_t)t);
        atomicOr(&lds[w0 + 1], (uint32_t)(t >> 32));
      }
    };
    // One window row's channels, as far as they belong to this copy.  The copies of a level share
    // the channels out in turn (channel c goes to copy c mod copies), so the low bits of a tile
    // channel's code follow from the copy and the high bits from the trip: with the number of
    // copies known at compile time, which planes a channel wants set costs one select per low bit,
    // once, and nothing per channel.
    const bool border = a.pad_mode == kPadBorder;
    auto row_channels = [&](auto lc_tag, int off, BW in_row, BW pad_row, BW fz_row) {
      constexpr int LC = decltype(lc_tag)::value, COPIES = 1 << LC;
      BW low = in_row;
#pragma unroll
      for (int k = 0; k < LC && k < PR::P; ++k) low &= ((sl.copy >> k) & 1) ? wp[k] : (BW)~wp[k];
#pragma unroll
      for (int j = 0; j * COPIES < PR::K; ++j) {
        BW bits = low;
#pragma unroll
        for (int k = LC; k < PR::P; ++k) bits &= ((j >> (k - LC)) & 1) ? wp[k] : (BW)~wp[k];
        if (j * COPIES <= 1 && 1 < (j + 1) * COPIES)  // the wall channel doubles as padding
          bits |= (!border && sl.copy == 1 - j * COPIES) ? pad_row : (BW)0;
        const bool mine = (j + 1) * COPIES <= PR::K || j * COPIES + sl.copy < PR::K;
        // (no test for an empty row: with a window of any size some lane of the wavefront nearly
        // always has a tile of the kind, so the test only skipped work lane by lane, which costs
        // the same as doing it: measured, 64x64 maze 15.37 -> 15.13 us per step, 32x32 dungeon
        // 13.3 -> 12.9)
        if (mine) emit(off + j * COPIES * cstride, bits);
      }
      if (border && sl.copy == (PR::K & (COPIES - 1)) && pad_row != 0)
        emit(off + (PR::K - sl.copy) * cstride, pad_row);
      if (a.obs_frozen_channel && sl.copy == (Cfz & (COPIES - 1)) && fz_row != 0)
        emit(off + (Cfz - sl.copy) * cstride, fz_row);
    };
    auto row_channels_any = [&](int off, BW in_row, BW pad_row, BW fz_row) {
      if (sl.copies_log2 == 0) {
        row_channels(std::integral_constant<int, 0>{}, off, in_row, pad_row, fz_row);
      } else if constexpr (LEAN && S <= 32) {
        if (sl.copies_log2 == 1) row_channels(std::integral_constant<int, 1>{}, off, in_row, pad_row, fz_row);
        if constexpr (S == 16) {
          if (sl.copies_log2 == 2) row_channels(std::integral_constant<int, 2>{}, off, in_row, pad_row, fz_row);
        }
      } else {
        // the general form: the channel's code is looked at bit by bit at run time
        for (int c = sl.copy; c < C; c += sl.copies, off += sl.copies * cstride) {
          BW bits = c < PR::K ? in_row : (BW)0;
#pragma unroll
          for (int k = 0; k < PR::P; ++k) bits &= ((c >> k) & 1) ? wp[k] : (BW)~wp[k];
          bits |= c == padc ? pad_row : (BW)0;
          if (c == Cfz) bits = fz_row;
          if (bits != 0) emit(off, bits);
        }
      }
    };
    if constexpr (S == 16) {
      // A 16-row buffer fills half of a typical window: every lane has rows above or below the
      // buffer to write, and those show nothing but padding.  Two passes (measured: 2-6 % ahead of
      // one loop over all rows and channels here, behind it for the larger buffers).
      // (a) the lane's own row of the buffer, if the window shows it
      const int i_own = L.y - y0;
      if (i_own >= 0 && i_own < ow) row_channels_any(pl.lane_off + i_own * ow, win_in, out_win, win_fz);
      // (b) window rows above or below the buffer: only the padding channel shows them; the copy
      // that owns that channel writes them, the rows dealt out over its lanes
      if ((padc & (sl.copies - 1)) == sl.copy) {
        const int off_pad = pl.lane_off + ((padc >> sl.copies_log2) << sl.copies_log2) * cstride;
        for (int i = i_own & (S - 1); i < ow; i += S)
          if (i != i_own) emit(off_pad + i * ow, owmask);
      }
    } else {
      for (int i = (L.y - y0) & (S - 1); i < ow; i += S) {
        const bool real = (y0 + i) == L.y;  // otherwise the row lies above or below the buffer
        row_channels_any(pl.lane_off + i * ow, real ? win_in : (BW)0, real ? out_win : owmask,
                         real ? win_fz : (BW)0);
      }
    }
  }
  lds_sync();

  if (a.obs_packed) {
    // bit-packed format: the stream itself is the output, 128 bits per aligned 16-byte chunk
    const uint4* lds128 = reinterpret_cast<const uint4*>(lds);
    for (int q = pl.q_lo + L.lane; q < pl.q_hi; q += 64) {
      const uint4 v = lds128[q];
      const u32x4 nv = {v.x, v.y, v.z, v.w};
      *(global_u32x4*)(pl.base + ((uint32_t)q << 4)) = nv;
    }
    if (pl.edge_want) *(global_u8*)(pl.base + pl.edge_pos) = reinterpret_cast<const uint8_t*>(lds)[pl.edge_pos];
    return;
  }
  const uint16_t* lds16 = reinterpret_cast<const uint16_t*>(lds);
  auto widen = [&](uint32_t b) {
    uint4 v;
    v.x = __umul24(b & 15u, 0x00204081u) & 0x01010101u;
    v.y = __umul24((b >> 4) & 15u, 0x00204081u) & 0x01010101u;
    v.z = __umul24((b >> 8) & 15u, 0x00204081u) & 0x01010101u;
    v.w = __umul24(b >> 12, 0x00204081u) & 0x01010101u;
    return v;
  };
  // chunks that lie completely inside the region: no bounds test, one aligned 16-byte store each
  if (a.stream_obs == kStoreThrough) {
    // Agent-scope stores: the L2 passes them on at once instead of keeping the lines dirty until
    // the write-back at the end of the kernel, which would otherwise follow the last wavefront
    // and cost about as long as the stores themselves.  (The compiler has no builtin for a
    // 16-byte store with a scope; nothing in the kernel reads these bytes back.)
    for (int q = pl.q_lo + L.lane; q < pl.q_hi; q += 64) {
      const uint4 v = widen(lds16[q]);
      u32x4 nv = {v.x, v.y, v.z, v.w};
      // (the s_nop: a store of more than 64 bits needs one wait state before a vector instruction
      // may overwrite its data registers, and the compiler does not look inside the asm string)
      asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 0" ::"v"(pl.base + ((uint32_t)q << 4)), "v"(nv));
    }
  } else if (a.stream_obs == kStoreStream) {
    // far more than the last-level cache holds: stream the bytes past it
    for (int q = pl.q_lo + L.lane; q < pl.q_hi; q += 64) {
      const uint4 v = widen(lds16[q]);
      u32x4 nv = {v.x, v.y, v.z, v.w};
      __builtin_nontemporal_store(nv, (global_u32x4*)(pl.base + ((uint32_t)q << 4)));
    }
  } else {
    for (int q = pl.q_lo + L.lane; q < pl.q_hi; q += 64) {
      const uint4 v = widen(lds16[q]);
      const u32x4 nv = {v.x, v.y, v.z, v.w};
      *(global_u32x4*)(pl.base + ((uint32_t)q << 4)) = nv;
    }
  }
  // the partial chunk at the head (lanes 0-15, one byte each) and at the tail (lanes 16-31)
  if (pl.edge_want)
    *(global_u8*)(pl.base + pl.edge_pos) = (uint8_t)((lds16[pl.edge_pos >> 4] >> (pl.edge_pos & 15)) & 1u);
}

// ------------------------------------------------------------------ kernels

template <int S, int PROBLEM>
__device__ __forceinline__ void store_metrics(int32_t* dst, const int (&m)[Prob<PROBLEM>::M]) {
  constexpr int M = Prob<PROBLEM>::M;
  int4* v = reinterpret_cast<int4*>(dst);
#pragma unroll
  for (int q = 0; q < (M + 3) / 4; ++q) {
    int4 t;
    t.x = 4 * q + 0 < M ? m[4 * q + 0] : 0;
    t.y = 4 * q + 1 < M ? m[4 * q + 1] : 0;
    t.z = 4 * q + 2 < M ? m[4 * q + 2] : 0;
    t.w = 4 * q + 3 < M ? m[4 * q + 3] : 0;
    v[q] = t;
  }
}

// Workgroups are handed to the eight accelerator dies (each with an L2 of its own) in turn, so
// workgroups b and b + 1 never share an L2, while the output regions of neighbouring level groups
// share the cache line on which one ends and the next begins (an observation is seldom a multiple
// of 128 bytes).  Written through two L2s, such a line reaches memory as two partial writes, and
// measured on plain stores that costs a quarter to a half of the write rate (regions of 9610 bytes:
// 4.2 against 5.6 TB/s; of 1922 bytes: 3.2 against 6.3).  So die x takes a contiguous run of level
// groups: the blocks b = x, x + 8, x + 16, ... work on consecutive groups, and both halves of a
// shared line meet in one L2.  A bijection on 0 .. n-1 for every n.  Used by rollouts that store
// with ordinary stores (maze16 at a batch of 65 536: +12 % steps per second, binary16 +7 %, maze64
// and binary32 with the 63-cell window +6 %; with non-temporal stores, which do not wait in the L2,
// it costs the dungeon 4 %).  A launch per step is better off with blocks in their natural order,
// whatever the store kind (measured: maze16 6.2 against 5.7 us, maze64 18.1 against 17.1): blocks
// that run at the same time then write neighbouring addresses.
template <bool ROLLOUT> __device__ __forceinline__ int level_group_of_block(int by_die) {
  const int b = (int)blockIdx.x, n = (int)gridDim.x;
  if constexpr (!ROLLOUT) return b;
  const int x = b & 7, q = n >> 3, rem = n & 7;
  return by_die ? x * q + min(x, rem) + (b >> 3) : b;
}

// Which wavefront, which levels: shared prologue of the two kernels.
template <int S> struct WaveMap {
  int wave, env0, nvalid, env, envl;
  bool valid, primary;
  Slot sl;
  uint32_t* lds;
  // Wavefront number `wave_` of a launch whose wavefronts hold 1 << lg_ levels each.  (Without a
  // split there is one workgroup per wavefront's worth of levels and exactly that many workgroups.)
  __device__ __forceinline__ void init(const KArgs& a, const Lanes<S>& L, uint32_t* lds_, int wave_, int lg_) {
    constexpr int G = 64 / S;
    wave = wave_;
    lds = lds_;
    const int lg = G == 1 ? 0 : lg_;  // levels per wavefront = 1 << lg
    const int epw = 1 << lg;
    sl.copies = G >> lg;
    sl.copies_log2 = (G == 4 ? 2 : G == 2 ? 1 : 0) - lg;
    sl.slot = L.g & (epw - 1);
    sl.copy = L.g >> lg;
    env0 = wave << lg;
    nvalid = min(epw, a.B - env0);
    env = env0 + sl.slot;
    valid = env < a.B;
    primary = valid && sl.copy == 0;
    envl = valid ? env : min(env0, a.B - 1);  // an index that is always safe to load from
  }
};

// WIDTH: a kernel that is launched only for windows of up to 32 cells (kWidthNarrow) or only for
// wider ones (kWidthWide) carries one of the two forms of the code; the registers of the wide
// form, whose window rows are 64-bit, otherwise set the kernel's occupancy for everybody.
constexpr int kWidthAny = 0, kWidthNarrow = 1, kWidthWide = 2;
template <int S, int PROBLEM, bool CLEARED = false, bool LEAN = false, int WIDTH = kWidthAny>
__device__ __forceinline__ void observe(const KArgs& a, const Lanes<S>& L, const WaveMap<S>& wm,
                                        const ObsPlan& pl,
                                        const typename RowWord<S>::T (&p)[Prob<PROBLEM>::P],
                                        typename RowWord<S>::T fz, typename RowWord<S>::T inside,
                                        int qy, int qx) {
  if (WIDTH == kWidthWide || (WIDTH == kWidthAny && a.obs_w > 32))
    write_obs<S, PROBLEM, true, CLEARED, LEAN>(a, L, wm.sl, pl, wm.lds, p, fz, inside, qy, qx);
  else
    write_obs<S, PROBLEM, false, CLEARED, LEAN>(a, L, wm.sl, pl, wm.lds, p, fz, inside, qy, qx);
}

// Reset / observe: either a fresh episode 0 from the seed, with its metrics and the default targets, or
// the stored level; then its observation, if a buffer is given.
template <int S, int PROBLEM>
__global__ __launch_bounds__(64) void init_kernel(KArgs a) {
  using W = typename RowWord<S>::T;
  using PR = Prob<PROBLEM>;
  extern __shared__ __align__(16) uint32_t lds_all[];
  Lanes<S> L;
  WaveMap<S> wm;
  wm.init(a, L, lds_all, level_group_of_block<false>(0), a.envs_per_wave_log2 & 0xff);
  W* planes = reinterpret_cast<W*>(a.planes);
  W* frozen = reinterpret_cast<W*>(a.frozen);
  const size_t ridx = (size_t)wm.envl * S + L.y;

  W p[PR::P], fz;
  int h, w, py, px;
  EnvRec er;
  if (a.fresh) {
    er.key = env_key(a.seed, (uint64_t)wm.envl, 0);
    er.t = 0;
    er.n_changes = 0;
    er.episode = 0;
    er.pad_ = 0;
    begin_episode<S, PROBLEM>(a, L, er.key, p, fz, h, w, py, px);
    er.cell_frozen = L.gany(L.y == py && ((fz >> px) & 1)) ? 1u : 0u;
    er.h = (uint8_t)h;
    er.w = (uint8_t)w;
    er.py = (uint8_t)py;
    er.px = (uint8_t)px;
    if (wm.primary) {
#pragma unroll
      for (int i = 0; i < PR::P; ++i) planes[(size_t)i * a.plane_stride + ridx] = p[i];
      frozen[ridx] = fz;
      if (L.y == 0) a.env[wm.env] = er;
    }
  } else {
    er = a.env[wm.envl];
    h = er.h;
    w = er.w;
    py = er.py;
    px = er.px;
#pragma unroll
    for (int i = 0; i < PR::P; ++i) p[i] = planes[(size_t)i * a.plane_stride + ridx];
    fz = 0;
    if (a.obs_frozen_channel) fz = frozen[ridx];
  }
  const W inside = inside_row<W>(L.y, h, w);
  if (a.fresh) {
    int m[PR::M];
    W comp;
    full_metrics<S, PROBLEM>(L, p, inside, wm.valid, m, comp);
    if (wm.primary && L.y == 0) store_metrics<S, PROBLEM>(a.metrics + (size_t)wm.env * kMaxMetrics, m);
    if constexpr (PROBLEM == kBinary) {  // (the plane after the tile planes)
      if (wm.primary) planes[(size_t)PR::P * a.plane_stride + ridx] = comp;
    }
    if (wm.primary && L.y < PR::M) {
      uint32_t t = pack_range(a.target_lo[L.y], a.target_hi[L.y]);
      if ((a.ctrl_mask >> L.y) & 1u) t = control_target(a, er.key, L.y);
      a.targets[(size_t)wm.env * kMaxMetrics + L.y] = t;
    }
  }
  if (a.obs != nullptr)
    observe<S, PROBLEM>(a, L, wm, obs_plan(a, L.lane, wm.sl, a.obs, wm.env0, wm.nvalid), p, fz, inside, py, px);
}

// The sweep above where a wavefront has one level only: all its lanes are at the same layer, so that nothing
// but the last layers has to be kept: a layer is its own 10 vector instructions and a quarter of a comparison, where
// the other form adds some 8 to it (exact diameter of 1024 random 64x64 levels 66.9 -> 50.8 us, with the ball's).
// A step, which sweeps seldom and not far, is no faster with it (4096 64x64 binary levels 8.70 / 8.96 us).
__device__ __forceinline__ int sweep_alone(const Lanes<64>& L, uint64_t seed, uint64_t pass, uint64_t& last, uint64_t& comp) {
  constexpr int S = 64;
  uint64_t V = seed, before = seed;  // the last layer, and the one before it
  int k = 0;
  for (int n = 0; n < kShortTrips; ++n) {
    const uint64_t one = L.grow(V, pass), two = L.grow(one, pass);
    if (!wave_any<S>(two != one)) {  // a second layer that adds nothing means the flood is complete
      const bool odd = wave_any<S>(one != V);
      comp = one;
      last = odd ? one & ~V : k == 0 ? seed : V & ~before;
      return odd ? k + 1 : k;
    }
    before = one;
    V = two;
    k += 2;
  }
  for (;; k += 4) {
    const uint64_t one = L.grow(V, pass), two = L.grow(one, pass), three = L.grow(two, pass), four = L.grow(three, pass);
    if (!wave_any<S>(four != three)) {
      comp = three;
      last = three & ~two;
      if (wave_any<S>(last != 0)) return k + 3;
      last = two & ~one;
      if (wave_any<S>(last != 0)) return k + 2;
      last = one & ~V;
      if (wave_any<S>(last != 0)) return k + 1;
      last = V & ~before;
      return k;
    }
    before = three;
    V = four;
  }
}

template <int S>
__device__ __forceinline__ int exact_sweep(const Lanes<S>& L, typename RowWord<S>::T seed, typename RowWord<S>::T pass,
                                           typename RowWord<S>::T& last, typename RowWord<S>::T& comp) {
  if constexpr (S == 64) return sweep_alone(L, seed, pass, last, comp);
  else return sweep<S>(L, seed, pass, last, comp);
}

// The cells within r edges of a seed (r the same in every lane of a group), and in `ring` those
// exactly r edges away.
template <int S>
__device__ __forceinline__ typename RowWord<S>::T ball(const Lanes<S>& L, typename RowWord<S>::T seed, typename RowWord<S>::T pass,
                                                       int r, typename RowWord<S>::T& ring) {
  using W = typename RowWord<S>::T;
  W V = seed, inner = 0;
  if constexpr (S == 64) {  // (one level to a wavefront: all lanes are at the same layer)
    const int n = wave_any<S>(seed != 0) ? __builtin_amdgcn_readfirstlane(r) : 0;
    for (int i = 0; i < n; ++i) {
      inner = V;
      V = L.grow(V, pass);
    }
    ring = V & ~inner;
    return V;
  }
  for (int i = 0; wave_any<S>(i < r && seed != 0); ++i) {
    const W grown = L.grow(V, pass);
    inner = i < r ? V : inner;
    V = i < r ? grown : V;
  }
  ring = V & ~inner;
  return V;
}

// A cell of a set near the middle of its rows, and of the columns of that row.
template <int S>
__device__ __forceinline__ typename RowWord<S>::T middle_cell(const Lanes<S>& L, typename RowWord<S>::T set) {
  using W = typename RowWord<S>::T;
  // the highest set bit at or below the middle between the lowest and the highest one
  auto middle = [](uint64_t v) { return 63 - __builtin_clzll(v & (~0ull >> (63 - (__builtin_ctzll(v) + 63 - __builtin_clzll(v)) / 2))); };
  const uint64_t rows = L.gbits(__builtin_amdgcn_ballot_w64(set != 0));
  if (rows == 0 || L.y != middle(rows)) return 0;
  return (W)1 << middle((uint64_t)set);
}

// The side n of the largest square that no shortest path of more than `best` edges fits into.  Such a
// path never fills a 2 x 2 square, so that an n x n square holds at most 3 n^2 / 4 of its cells for
// even n, and for odd n as many as the square of side n - 1 and the 2 n - 1 cells around it.
__device__ __forceinline__ int square_below(int best) {
  constexpr int kEdges[] = {2, 7, 11, 20, 26, 39, 47, 64, 74, 95, 107, 132, 146, 175, 191};  // n = 2, 3, ... 16
  int n = 1;
#pragma unroll
  for (int i = 0; i < 15; ++i) n += best >= kEdges[i] ? 1 : 0;
  return n;
}

// The cells of `todo`, a union of whole components, whose components fit into a square of side n
// (n > 1) of the grid moved by (my, mx): those that a flood from the cells next to a grid line which
// their component crosses does not reach.
template <int S>
__device__ __forceinline__ typename RowWord<S>::T inside_squares(const Lanes<S>& L, typename RowWord<S>::T todo, int n, int my, int mx) {
  using W = typename RowWord<S>::T;
  uint64_t lines = 0;
  for (int x = 0; x < S; x += n) lines |= 1ull << x;
  W down = todo & L.from_above(todo);  // (not inside a condition: a lane shift reads active lanes only)
  if (((lines << my) >> L.y & 1) == 0) down = 0;
  const W across = todo & (W)(todo << 1) & (W)(lines << mx);
  W last, reached;
  exact_sweep<S>(L, down | across, todo, last, reached);
  return todo & ~reached;
}

// The cells of `todo`, a union of whole components, whose components fit into a square of side 16 of the grid
// moved by (my, mx), each 0 or 8, that holds no more than best + 1 cells of such components: no path in it has
// more than `best` edges.  (A square that the move cuts in two counts as one.)
template <int S>
__device__ __forceinline__ typename RowWord<S>::T inside_few(const Lanes<S>& L, typename RowWord<S>::T todo, int best, int my, int mx) {
  using W = typename RowWord<S>::T;
  static_assert(S >= 32, "a square is a row of 16 lanes");
  const W in = inside_squares<S>(L, todo, 16, my, mx);
  // rows and columns moved so that squares are whole lane rows and whole pieces of a word, and back
  auto turned = [](W r, int by) -> W { return (W)((W)(r >> by) | (W)((W)(r << 1) << (S - 1 - by))); };
  const W v = turned(L.gread(in, (L.y + my) & (S - 1)), mx);
  W keep = 0;
#pragma unroll
  for (int q = 0; q < S; q += 32) {
    const uint32_t two = (uint32_t)(v >> q);  // rows of two squares
    int c = popc(two & 0xffffu) | popc(two >> 16) << 16;
    c += __builtin_amdgcn_update_dpp(0, c, 0xB1, 0xf, 0xf, false);  // sums over 2, 4, 8 and 16 lanes
    c += __builtin_amdgcn_update_dpp(0, c, 0x4E, 0xf, 0xf, false);
    c += __builtin_amdgcn_update_dpp(0, c, 0x141, 0xf, 0xf, false);
    c += __builtin_amdgcn_update_dpp(0, c, 0x140, 0xf, 0xf, false);
    keep |= (W)(((c & 0xffff) <= best + 1 ? 0xffffu : 0u) | ((c >> 16) <= best + 1 ? 0xffff0000u : 0u)) << q;
  }
  return in & L.gread(turned(keep, (S - mx) & (S - 1)), (L.y - my) & (S - 1));
}

// Exact diameter: the longest shortest path between two cells of a level.  Components are taken one
// after the other, and of a component's cells only those that a longer path than the best so far
// could start from are swept:
//  * a sweep from any cell (eccentricity e) finishes a component with 2 e <= best;
//  * otherwise two sweeps find the two ends of a long path and a third one starts from its middle c:
//    two cells further apart than `best` are not both within best / 2 of c, so that only the cells
//    outside that ball are left, the rim: a few on random maps, half of the cells on a long loop;
//  * a sweep from a cell v of eccentricity e(v) rules out every cell u with d(u, v) + e(v) <= best.
// The first component a wavefront takes is the one in which a flood from a row arrives last, most
// often a large one; with `best` that large nearly all others end after their first sweep, or, being
// small, before it (inside_squares).
// A workgroup is 1 << waves_log2 wavefronts on the same levels, each with a part of their rows (as has
// each copy of a level inside a wavefront), which take components from their own rows first and then
// from all.  What is left to do, and the best so far, they share through LDS: a component belongs to
// the part that takes its first cell out of the shared set.  Its owner sweeps a few rim cells itself
// (each rules out many of the others, so that all parts together would sweep in vain), and what is left
// of all rims is shared out cell by cell once nobody has a component left.  Lane groups work at their
// own pace (a group that has nothing to do in a sweep has no seed); every loop ends because each turn
// takes cells out of a finite set.
// 1420 flood layers in 66 floods for a random 64x64 level of 50 % walls (1890 in 101 before inside_few, and while a
// part told the others its finds only once it was done with a component), bound by the latency of one after the other
// in small batches and by that and vector instructions (60 % of the issue slots) from 1024 levels on: a sweep from each of its 2000 open cells instead took 1350 us for 1024 levels (a launch of 4096
// wavefronts and one that folded their results); this takes 51 (76.9 before inside_few and sweep_alone).  A loop of 2080 cells
// is the worst there is, 1040 sweeps of 1040 layers and bound by instructions: 64 such levels 5.9 ms
// (37.8 while the owner swept the whole rim, 6.5 from each cell on 4096 wavefronts; one level alone takes
// as long here, and took 2.0 there), 1024 of them 22.5 ms (38.0, 104).
// (Of 0, 2, 4, 8 and 16 own rim cells: 1024 levels of rooms 68, 67, 57, 57, 57 us, of a grid of corridors 63,
// 78, 77, 107, 114.)
constexpr int kOwnRimCells = 4;
template <int S, int PROBLEM>
__global__ __launch_bounds__(1024) void exact_diameter_kernel(KArgs a, int32_t* out, int waves_log2) {
  using W = typename RowWord<S>::T;
  using PR = Prob<PROBLEM>;
  constexpr int kWords = sizeof(W) / 4;
  // sets of cells that the wavefronts share, [slot * S + y]: those of the components nobody has taken
  // yet, those still to be swept, and the middles of the components these lie in
  __shared__ uint32_t left[kWords][64], rim[kWords][64], middles[kWords][64];
  __shared__ int shared_best[64 / S], any_rim;
  Lanes<S> L;
  WaveMap<S> wm;
  wm.init(a, L, nullptr, (int)blockIdx.x, a.envs_per_wave_log2 & 0xff);
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int part = (wave << wm.sl.copies_log2) + wm.sl.copy, parts_log2 = waves_log2 + wm.sl.copies_log2;
  const W* planes = reinterpret_cast<const W*>(a.planes);
  const size_t ridx = (size_t)wm.envl * S + L.y;
  W p[PR::P];
#pragma unroll
  for (int i = 0; i < PR::P; ++i) p[i] = planes[(size_t)i * a.plane_stride + ridx];
  const uint32_t hw = *reinterpret_cast<const uint32_t*>(a.env + wm.envl);
  const int h = (int)(hw & 0xffu), w = (int)((hw >> 8) & 0xffu);
  const W inside = wm.valid ? inside_row<W>(L.y, h, w) : (W)0;
  const W pass = inside & ~channel_row<PROBLEM, W>(p, inside, 1);
  // (a cell on its own is the end of no path)
  W todo = pass & ((W)(pass << 1) | (W)(pass >> 1) | L.from_above(pass) | L.from_below(pass));
  const int row = wm.sl.slot * S + L.y;
  if (wave == 0 && wm.sl.copy == 0) {
#pragma unroll
    for (int k = 0; k < kWords; ++k) {
      left[k][row] = (uint32_t)((uint64_t)todo >> (32 * k));
      rim[k][row] = middles[k][row] = 0;
    }
    if (L.y == 0) shared_best[wm.sl.slot] = any_rim = 0;
  }
  __syncthreads();
  using Shared = uint32_t (&)[kWords][64];
  auto take = [&](Shared set, W cells) -> W {  // out of a shared set; returns what it held of them
    W had = (W)atomicAnd(&set[0][row], ~(uint32_t)cells);
    if constexpr (kWords == 2) had |= (W)atomicAnd(&set[1][row], ~(uint32_t)((uint64_t)cells >> 32)) << 32;
    return had & cells;
  };
  auto put = [&](Shared set, W cells) {
    atomicOr(&set[0][row], (uint32_t)cells);
    if constexpr (kWords == 2) atomicOr(&set[1][row], (uint32_t)((uint64_t)cells >> 32));
  };
  auto look = [&](Shared set) -> W {
    W v = (W)__hip_atomic_load(&set[0][row], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    if constexpr (kWords == 2)
      v |= (W)__hip_atomic_load(&set[1][row], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) << 32;
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");  // (with the release below: every look is acted on)
    return v;
  };
  auto best_so_far = [&]() {
    return __hip_atomic_load(&shared_best[wm.sl.slot], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  };
  const int row_lo = part * h >> parts_log2, row_mid = (2 * part + 1) * h >> (parts_log2 + 1);
  auto choose = [&](W set) -> W {  // a cell, from this part's rows on if there is one
    const W mine = first_cell<S>(L, L.y >= row_lo ? set : (W)0), any = first_cell<S>(L, set);
    return L.gany(mine != 0) ? mine : any;
  };
  int best = 0, side = 1;
  W none, comp;
  // Sweeps a rim cell and returns the cells that no longer path than the best starts from by what it
  // found: a new best widens the ball around the middle of the component, otherwise v's own ball goes.
  auto rule_out = [&](W v, W middle) -> W {
    W far, all;
    const int e = exact_sweep<S>(L, v, pass, far, all);
    const bool longer = e > best;
    best = max(best, e);
    return ball<S>(L, longer ? middle & all : v, pass, longer ? best >> 1 : best - e, none);
  };
  W src;
  {
    W cross = L.y == row_mid ? todo : (W)0;
    if (parts_log2 == 0) cross |= todo & ((W)1 << (w / 2));
    exact_sweep<S>(L, cross, todo, src, comp);
    src = first_cell<S>(L, src);
  }
  for (bool first = true;; first = false) {
    todo = look(left);
    best = max(best, best_so_far());
    if (!first) {
      const int n = square_below(best);
      if (wave_any<S>(n > side)) {  // (once, and again should `best` grow by much later on)
        for (int turn = 0; turn < max(4 >> parts_log2, 1); ++turn) {  // (four grids at least)
          const int t = part + (turn << parts_log2);
          const int half = n >> 1, quarter = (t >> 2) & 1 ? n >> 2 : 0;
          W small = inside_squares<S>(L, n > side ? todo : (W)0, max(n, 2), ((t & 1) ? half : 0) + quarter,
                                            (((t ^ (t >> 1)) & 1) ? half : 0) + quarter);
          take(left, small);
          todo &= look(left);
          if constexpr (S > 16) {
            small = inside_few<S>(L, n > side ? todo : (W)0, best, (t & 1) ? 8 : 0, ((t ^ (t >> 1)) & 1) ? 8 : 0);
            take(left, small);
            todo &= look(left);
          }
        }
        side = max(side, n);
      }
    }
    if (!first || !L.gany(src != 0)) src = choose(todo);
    if (!wave_any<S>(src != 0)) break;
    W far;
    const int e1 = exact_sweep<S>(L, src, pass, far, comp);
    // (the first cell decides, before the others go: a part that looks while they do sees a piece of
    // the component, which it may take for a small one but no longer for its own.  The words of a row
    // and the rows are atomics of their own, hence the fence: were the others seen to go first, a piece
    // that still holds the first cell could be dropped as a small component and belong to nobody)
    const bool ours = L.gany(take(left, first_cell<S>(L, comp)) != 0);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    take(left, comp);
    // (told to the others at once: a component no more than half as deep as another is done with)
    if (L.y == 0) atomicMax(&shared_best[wm.sl.slot], e1);
    best = max(best, best_so_far());
    bool open = ours && 2 * e1 > best;
    if (wave_any<S>(open)) {
      W end_a = first_cell<S>(L, far);
      if (!open) end_a = 0;
      const int e2 = exact_sweep<S>(L, end_a, pass, far, none);
      if (L.y == 0) atomicMax(&shared_best[wm.sl.slot], e2);
      best = max(best, best_so_far());
      open = open && 2 * e1 > best;
      if (wave_any<S>(open)) {
        W ring_a, ring_b;
        W end_b = first_cell<S>(L, far);
        if (!open) end_a = end_b = 0;
        ball<S>(L, end_a, pass, e2 >> 1, ring_a);
        ball<S>(L, end_b, pass, e2 - (e2 >> 1), ring_b);
        const W centre = middle_cell<S>(L, ring_a & ring_b);
        const int ec = exact_sweep<S>(L, centre, pass, far, none);
        best = max(best, ec);
        open = open && 2 * ec > best;
        const W core = open ? centre : (W)0;
        const W near = ball<S>(L, core, pass, best >> 1, none);
        W mine = open ? comp & ~near : (W)0;
        for (int turn = 0; turn < kOwnRimCells; ++turn) {
          const W v = first_cell<S>(L, mine);
          if (!wave_any<S>(v != 0)) break;
          mine &= ~v;
          mine &= ~rule_out(v, core);
        }
        if (wave_any<S>(mine != 0)) {
          put(rim, mine);
          put(middles, core);
          any_rim = 1;
        }
      }
      if (L.y == 0) atomicMax(&shared_best[wm.sl.slot], best);
    }
  }
  if (L.y == 0) atomicMax(&shared_best[wm.sl.slot], best);
  __syncthreads();
  // What is left of the rims, shared out cell by cell: on a level with a long loop, all of whose cells
  // are equally far from their farthest one, that is half of its cells, each with a sweep of its own.
  if (any_rim) {
    for (;;) {
      W v = 0;
      for (;;) {  // (another part may be quicker; each turn some part gets a cell)
        const W c = choose(L.gany(v != 0) ? (W)0 : look(rim));
        if (!wave_any<S>(c != 0)) break;
        v |= take(rim, c);
      }
      if (!wave_any<S>(v != 0)) break;
      best = max(best, best_so_far());
      const int before = best;
      take(rim, rule_out(v, look(middles)));
      if (best > before && L.y == 0) atomicMax(&shared_best[wm.sl.slot], best);
    }
    __syncthreads();
  }
  if (wave == 0 && wm.primary && L.y == 0) out[wm.env] = shared_best[wm.sl.slot];
}

// What a modifying edit does to the metrics that have to be searched for.  `regions`: by how much the
// region count changes, or the new count in recount mode; `searched`: whether path (and enemy) are the
// new values, otherwise they are as before.  Binary problem: `comp`, the component of the first
// walkable cell before the edit if `comp_known`, becomes that after it.  (p, inside: the level after the
// edit; nothing is asked of a level that did not change.)
// For the relay's searchers; step_body has the same written out, in a form that updates the vector where
// something was found: called from there this form took steps of 262 144 16x16 binary levels from 101.5 to
// 103.6 us, whether it returned its results or handed them on inside the search's branch.
struct Moved {
  int regions, path, enemy;
  bool searched;
};
template <int S, int PROBLEM>
__device__ __forceinline__ Moved after_edit(bool recount, const Lanes<S>& L, const typename RowWord<S>::T (&p)[Prob<PROBLEM>::P],
                                            typename RowWord<S>::T inside, bool changed, int old_code, int act, int h, int w,
                                            int py, int px, typename RowWord<S>::T& comp, bool comp_known) {
  using W = typename RowWord<S>::T;
  Moved mv = {0, 0, 0, false};
  const bool at_row = L.y == py;
  const W in = changed ? inside : (W)0;  // unchanged levels look empty: their loops end at once
  const W wall = channel_row<PROBLEM, W>(p, in, 1);
  const W pass = in & ~wall;
  const bool was_pass = old_code != 1, now_pass = act != 1;
  // regions
  if (recount) {
    mv.regions = regions_full<S>(L, pass, in, true);
  } else {
    const bool flip = changed && was_pass != now_pass;
    if (wave_any<S>(flip)) {
      const W cell = (flip && at_row) ? (W)1 << px : (W)0;
      int k;
      if constexpr (S == 16 && PROBLEM == kBinary) {  // (see neighbour_components)
        const W passw = flip ? (W)(pass & ~cell) : (W)0;
        k = neighbour_components<S>(L, (L.dilate(cell) & ~cell) & passw, passw);
      } else {
        k = components_around<S>(L, flip ? (W)(pass & ~cell) : (W)0, inside, cell, h, w, py, px);
      }
      if (flip) mv.regions = now_pass ? 1 - k : k - 1;
    }
  }
  // paths
  if constexpr (PROBLEM == kBinary) {
    // (every modifying edit of a binary level flips the walkability of its cell)
    const W cell = (changed && at_row) ? (W)1 << px : (W)0;
    const bool need = changed && !(comp_known && diameter_untouched<S>(L, comp, cell, L.dilate(cell), py, px, now_pass));
    if (wave_any<S>(need)) {
      W ncomp;
      const int dm = two_sweep_diameter<S>(L, need ? pass : (W)0, ncomp);
      if (need) {
        comp = ncomp;
        mv.path = dm;
      }
    }
    mv.searched = need;
  } else if constexpr (PROBLEM == kMaze) {
    W r;
    const int dd = nearest<S>(L, channel_row<PROBLEM, W>(p, in, 2), channel_row<PROBLEM, W>(p, in, 3), pass, r);
    mv.path = dd < 0 ? 0 : dd;
    mv.searched = changed;
  } else {
    // swapping empty and chest changes neither the graph nor any source or target set
    const bool plain = (old_code == 0 || old_code == 6) && (act == 0 || act == 6);
    const bool need = changed && !plain;
    if (wave_any<S>(need)) {
      const W inn = need ? in : (W)0;
      const W passn = need ? pass : (W)0;
      W k1, r;
      int d1, de;
      nearest_two<S>(L, channel_row<PROBLEM, W>(p, inn, 2), channel_row<PROBLEM, W>(p, inn, 3),
                     channel_row<PROBLEM, W>(p, inn, 5), passn, d1, k1, de);
      const int d2 = nearest<S>(L, k1, channel_row<PROBLEM, W>(p, inn, 4), passn, r);
      mv.path = (d1 >= 0 && d2 >= 0) ? d1 + d2 : 0;
      mv.enemy = de < 0 ? 0 : de;
    }
    mv.searched = need;
  }
  return mv;
}

// The observation wavefront of the split kernel: loads the level, applies the edit in registers
// (it stores nothing but the observation), finds the agent's next cell and writes the window
// around it.  It reads what the metrics wavefront of the same workgroup reads, and the workgroup
// barrier, which this wavefront enters only when its loads have returned, keeps that wavefront
// from storing the new state before.
template <int S, int PROBLEM, bool PIN, int WIDTH>
__device__ __forceinline__ void obs_wave_step(KArgs& a, const Lanes<S>& L, WaveMap<S>& wm, uint32_t* lds_all, int wid) {
  // (on entry `a` holds only what came in registers; the rest is fetched once the loads are issued)
  using W = typename RowWord<S>::T;
  using PR = Prob<PROBLEM>;
  if (wm.env0 >= a.B) {  // the batch ends inside this workgroup: only the barrier is owed
    __syncthreads();
    return;
  }
  const W* planes = reinterpret_cast<const W*>(a.planes);
  const size_t ridx = (size_t)wm.envl * S + L.y;
  W p[PR::P];
#pragma unroll
  for (int i = 0; i < PR::P; ++i) p[i] = planes[(size_t)i * a.plane_stride + ridx];
  // (with pinpoints their rows are loaded whether or not they are shown: no branch between the loads)
  W fz = 0;
  if constexpr (PIN) fz = reinterpret_cast<const W*>(a.frozen)[ridx];
  const uint4* erp = reinterpret_cast<const uint4*>(a.env + wm.envl);
  const uint4 er0 = erp[0], er1 = erp[1];
  const int act = a.actions[wm.envl];
  // where the observation goes is worked out, and its staging words are cleared, while the loads
  // are in flight (fenced off so that no use of a loaded value, with its wait, moves in between)
  __builtin_amdgcn_sched_barrier(0);
  fill_rest_of_args(a);
  wm.lds = lds_all + (wid - 1) * a.obs_lds_words;
  ObsPlan pl = obs_plan(a, L.lane, wm.sl, a.obs, wm.env0, wm.nvalid);
  obs_plan_pin(pl);
  obs_clear(wm.lds, L.lane, pl);
  __builtin_amdgcn_sched_barrier(0);
  // The barrier only once every load of the old state has returned: the metrics wavefront stores
  // the new state after it, and nothing else orders those stores behind these loads.  (That
  // wavefront requested the same words at the same time, so it would be waiting for them anyway.)
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  __builtin_amdgcn_sched_barrier(0);
  if (!PIN || !(a.use_frozen & 2)) fz = 0;

  int h = (int)(er0.x & 0xffu), w = (int)((er0.x >> 8) & 0xffu);
  const int py = (int)((er0.x >> 16) & 0xffu), px = (int)(er0.x >> 24);
  int t = (int)er0.y + 1;
  const uint64_t key = (uint64_t)er1.x | ((uint64_t)er1.y << 32);
  W inside = inside_row<W>(L.y, h, w);
  // the edit: writing the tile that is already there changes nothing, so the old tile is only
  // looked at when changes are counted against a budget
  const bool at_row = L.y == py;
  const bool may_write = wm.valid && act >= 0 && act < PR::K && er1.z == 0;
  bool done = t >= a.max_steps;
  if (a.max_changes > 0) {
    int old_code = 0;
#pragma unroll
    for (int i = 0; i < PR::P; ++i) old_code |= (L.gany(at_row && ((p[i] >> px) & 1)) ? 1 : 0) << i;
    const int n_changes = (int)er0.z + ((may_write && act != old_code) ? 1 : 0);
    done = done || n_changes >= a.max_changes;
  }
  if (may_write && at_row) {
#pragma unroll
    for (int i = 0; i < PR::P; ++i) p[i] = (p[i] & ~((W)1 << px)) | ((W)((act >> i) & 1) << px);
  }
  int qy = py, qx = px;
  if (a.pos_mode == kPosScan) {
    qx += 1;
    if (qx >= w) {
      qx = 0;
      qy += 1;
      if (qy >= h) qy = 0;
    }
  } else {
    uint64_t u = draw(key, 3, (uint32_t)t);
    qy = below((uint32_t)(u >> 32), h);
    qx = below((uint32_t)u, w);
  }
  const bool restart = wm.valid && done && a.autoreset != 0;
  if (wave_any<S>(restart)) {  // the observation then shows the first state of the next episode
    const KArgs& ra = cold_args<false>();
    W np[PR::P], nfz;
    int nh, nw, npy, npx;
    uint64_t nkey = env_key(ra.seed, (uint64_t)wm.envl, (uint64_t)((int)er0.w + 1));
    begin_episode<S, PROBLEM, true, kDrawsAbreast<S, PROBLEM, false>>(ra, L, nkey, np, nfz, nh, nw, npy, npx, restart, wm.envl);
    if (restart) {
#pragma unroll
      for (int i = 0; i < PR::P; ++i) p[i] = np[i];
      fz = nfz;
      inside = inside_row<W>(L.y, nh, nw);
      qy = npy;
      qx = npx;
    }
  }
  observe<S, PROBLEM, true, true, WIDTH>(a, L, wm, pl, p, fz, inside, qy, qx);
}

// Says that values have arrived: whatever loads them is waited for here and not, as the compiler would
// have it, at their first use inside a loop, where the wait would be one for everything that the
// loop's own stores have not finished yet, in every iteration.
template <typename T> __device__ __forceinline__ void arrived(T& v) {
  if constexpr (sizeof(T) == 8) {
    uint32_t lo = (uint32_t)v, hi = (uint32_t)((uint64_t)v >> 32);
    asm volatile("" : "+v"(lo), "+v"(hi));
    v = (T)(((uint64_t)hi << 32) | lo);
  } else {
    asm volatile("" : "+v"(v));
  }
}
template <typename T, typename... R> __device__ __forceinline__ void arrived(T& v, R&... rest) {
  arrived(v);
  arrived(rest...);
}

// The observation wavefront of a split rollout.  It needs nothing from the metrics wavefront: what
// an observation shows -- the edited level, the agent's next cell, a restarted episode -- follows
// from the loaded state, the seeds and the action stream alone, so this wavefront carries its own
// copy of the level through all the steps and only writes observations.  Where the batch leaves
// SIMDs idle, several such wavefronts take the steps in turn: this one writes the observations of
// the steps t with (t & turn_mask) == turn and only follows the level through the others.
// (TURNS = false is the same code for the launches in which every such wavefront writes every step: the
// test per step costs the large batches 7 % through the registers it ties up.  Each form has a kernel of
// its own: both in one, 65 536 32x32 binary levels with a 3-cell window took 22.2 us a step against 20.9.)
template <int S, int PROBLEM, bool TURNS>
__device__ __forceinline__ void obs_wave_rollout(const KArgs& a, const Lanes<S>& L, const WaveMap<S>& wm, int turn,
                                                 int turn_mask) {
  using W = typename RowWord<S>::T;
  using PR = Prob<PROBLEM>;
  if (wm.env0 >= a.B) {  // the batch ends inside this workgroup: only the barrier is owed
    __syncthreads();
    return;
  }
  const W* planes = reinterpret_cast<const W*>(a.planes);
  const size_t ridx = (size_t)wm.envl * S + L.y;
  W p[PR::P];
#pragma unroll
  for (int i = 0; i < PR::P; ++i) p[i] = planes[(size_t)i * a.plane_stride + ridx];
  W fz = reinterpret_cast<const W*>(a.frozen)[ridx];
  const uint4* erp = reinterpret_cast<const uint4*>(a.env + wm.envl);
  uint4 er0 = erp[0], er1 = erp[1];
  int act = a.actions[wm.envl];
  __builtin_amdgcn_sched_barrier(0);
  // (the metrics wavefront stores the final state only after this barrier, and the barrier comes
  // only after these loads have returned)
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int i = 0; i < PR::P; ++i) arrived(p[i]);
  arrived(fz, er0.x, er0.y, er0.z, er0.w, er1.x, er1.y, act);

  int h = (int)(er0.x & 0xffu), w = (int)((er0.x >> 8) & 0xffu);
  int py = (int)((er0.x >> 16) & 0xffu), px = (int)(er0.x >> 24);
  int t = (int)er0.y, n_changes = (int)er0.z, episode = (int)er0.w;
  uint64_t key = (uint64_t)er1.x | ((uint64_t)er1.y << 32);
  W inside = inside_row<W>(L.y, h, w);
  const int nsteps = a.rollout_steps;
  // Where an observation goes depends on its slot only through the slot's address modulo 16: with
  // slots a multiple of 16 bytes apart (any batch that is a multiple of 16, any layout padded to
  // cache lines) the plan is worked out once and only its base address moves from step to step.
  const size_t slot_bytes = (size_t)a.B * (size_t)a.env_obs_bytes;
  const bool fixed_plan = (slot_bytes & 15u) == 0;
  ObsPlan pl = obs_plan(a, L.lane, wm.sl, a.obs, wm.env0, wm.nvalid);
  uint8_t* const base0 = pl.base;
  int slot = 0;
  size_t slot_off = 0;
  for (int step = 0; step < nsteps; ++step) {
    int act_next = -1;
    if (step + 1 < nsteps) act_next = a.actions[(size_t)(step + 1) * a.B + wm.envl];
    // the edit (the old tile matters only when changes are counted against a budget)
    const bool at_row = L.y == py;
    const bool is_frozen = L.gany(at_row && ((fz >> px) & 1));
    const bool may_write = wm.valid && act >= 0 && act < PR::K && !is_frozen;
    t += 1;
    bool done = t >= a.max_steps;
    if (a.max_changes > 0) {
      int old_code = 0;
#pragma unroll
      for (int i = 0; i < PR::P; ++i) old_code |= (L.gany(at_row && ((p[i] >> px) & 1)) ? 1 : 0) << i;
      n_changes += (may_write && act != old_code) ? 1 : 0;
      done = done || n_changes >= a.max_changes;
    }
    if (may_write && at_row) {
#pragma unroll
      for (int i = 0; i < PR::P; ++i) p[i] = (p[i] & ~((W)1 << px)) | ((W)((act >> i) & 1) << px);
    }
    int qy = py, qx = px;
    if (a.pos_mode == kPosScan) {
      qx += 1;
      if (qx >= w) {
        qx = 0;
        qy += 1;
        if (qy >= h) qy = 0;
      }
    } else {
      uint64_t u = draw(key, 3, (uint32_t)t);
      qy = below((uint32_t)(u >> 32), h);
      qx = below((uint32_t)u, w);
    }
    const bool restart = wm.valid && done && a.autoreset != 0;
    if (wave_any<S>(restart)) {
      const KArgs& ra = cold_args<true>();
      W np[PR::P], nfz;
      int nh, nw, npy, npx;
      uint64_t nkey = env_key(ra.seed, (uint64_t)wm.envl, (uint64_t)(episode + 1));
      begin_episode<S, PROBLEM, true, kDrawsAbreast<S, PROBLEM, true>>(ra, L, nkey, np, nfz, nh, nw, npy, npx, restart, wm.envl);
      if (restart) {
#pragma unroll
        for (int i = 0; i < PR::P; ++i) p[i] = np[i];
        fz = nfz;
        h = nh;
        w = nw;
        inside = inside_row<W>(L.y, nh, nw);
        qy = npy;
        qx = npx;
        key = nkey;
        episode += 1;
        t = 0;
        n_changes = 0;
      }
    }
    if (!TURNS || (step & turn_mask) == turn) {
      if (fixed_plan) pl.base = base0 + slot_off;
      else pl = obs_plan(a, L.lane, wm.sl, a.obs + slot_off, wm.env0, wm.nvalid);
      observe<S, PROBLEM, false, true>(a, L, wm, pl, p, fz, inside, qy, qx);
    }
    slot = slot + 1 == a.obs_slots ? 0 : slot + 1;  // (step t writes slot t mod obs_slots)
    slot_off = slot == 0 ? 0 : slot_off + slot_bytes;
    py = qy;
    px = qx;
    act = act_next;
  }
}

// The sum over metrics, in index order, of weight * (old loss - new loss), in lane M - 1 of a lane group
// whose lane k holds metric k, its range and its weight: every lane its own term; then M-1 times every
// lane adds its term to what the lane before it holds, so that lane k ends with
// ((t[k-M+1] + ...) + t[k-1]) + t[k], terms before the first lane counting as zero.
template <int M> __device__ __forceinline__ float reward_of(int before, int after, uint32_t range, float weight) {
  const int lo = (int)(range & 0xffffu), hi = (int)(range >> 16);
  const int dl = loss(before, lo, hi) - loss(after, lo, hi);
  const float term = __fmul_rn(weight, (float)dl);
  float acc = __fadd_rn(0.0f, term);
#pragma unroll
  for (int j = 1; j < M; ++j) acc = __fadd_rn(__int_as_float((int)dpp_zero_fill<kRowShr1>((uint32_t)__float_as_int(acc))), term);
  return acc;
}

// ---- Relay: a rollout of a small batch.
// Its time is that of one dependent chain per step, and most of the machine is idle.  What the levels go
// through (edits, restarts, where the agent goes) does not depend on the metrics, and the searches of
// one step do not depend on those of another, so the wavefronts of a workgroup pass the steps of their
// levels on to each other, kRelaySteps at a time through LDS:
//   the leader    follows edits, counters, restarts and positions and writes them down;
//   the searchers apply the edits of all steps and work the metrics out for every n-th;
//   the observers do the same for the observations;
//   the adder     sums the rewards up from what the searchers found and keeps the metric vectors.
// While the leader is at one piece of the rollout, searchers and observers are at the piece before it and
// the adder at the one before that; one barrier a piece.  256-step rollouts of 64 levels, us per step,
// against one metrics wavefront and observation wavefronts that take turns: 16x16 binary 1.11 -> 0.62, 16x16
// maze 0.88 -> 0.53, 32x32 dungeon 1.22 -> 0.48, 64x64 maze 1.08 -> 0.56.  What is left is the observers'
// chain (without it 0.45 to 0.5) and the other wavefronts', none of which does much less.  Pieces of 8 steps
// keep the three stages short for rollouts of a few steps (4 steps of 64 dungeon levels 2.56 -> 2.12 us each),
// and give every searcher and observer two turns or more to even out.
template <int S, int PROBLEM> struct RelayTables {
  static constexpr int kLevels = 64 / S;  // of a workgroup, at most
  // what the leader wrote down of a step: x bits 0-2 the action, 3-5 the tile it replaced, 6 the level
  // changed, 7 the episode is done, 8 a new one begins; y the cell and the next one, a byte a number
  uint2 trace[3][kRelaySteps][kLevels];
  // what a searcher found (see Moved): x bit 0 path and enemy are new, bits 16-31 regions; y path | enemy << 16
  uint2 found[2][kRelaySteps][kLevels];
  // a new episode: its level (planes, pinpoints, height | width << 8) and its metrics; one a piece, since a
  // relay is run only for episodes of kRelaySteps steps or more
  typename RowWord<S>::T rows[3][kLevels][Prob<PROBLEM>::P + 1][S];
  int32_t hw[3][kLevels];
  int32_t metrics[2][kLevels][kMaxMetrics];
};
constexpr uint32_t kTraceChanged = 1u << 6, kTraceDone = 1u << 7, kTraceRestart = 1u << 8;
__device__ __forceinline__ int relay_pieces(int nsteps) { return (nsteps + kRelaySteps - 1) / kRelaySteps; }
// (LDS traffic of the pieces only: what a wavefront has stored to memory need not have arrived)
__device__ __forceinline__ void relay_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// The leader.  Lane y of a level's lane group prepares step y of a piece: the action, and (random
// positions) the cell the agent goes to after it, one hash for all the steps of all the levels.  The
// lane of the edited row alone knows the old tile, and writes the step down.
template <int S, int PROBLEM>
__device__ __forceinline__ void relay_leader(const KArgs& a, const Lanes<S>& L, const WaveMap<S>& wm, RelayTables<S, PROBLEM>& tables) {
  using W = typename RowWord<S>::T;
  using PR = Prob<PROBLEM>;
  static_assert(kRelaySteps <= 16, "a lane for every step of a piece");
  W* planes = reinterpret_cast<W*>(a.planes);
  W* frozen = reinterpret_cast<W*>(a.frozen);
  const size_t ridx = (size_t)wm.envl * S + L.y;
  W p[PR::P];
#pragma unroll
  for (int i = 0; i < PR::P; ++i) p[i] = planes[(size_t)i * a.plane_stride + ridx];
  W fz = frozen[ridx];
  const uint4* erp = reinterpret_cast<const uint4*>(a.env + wm.envl);
  uint4 er0 = erp[0], er1 = erp[1];
  const int nsteps = a.rollout_steps, pieces = relay_pieces(nsteps);
  auto action_of = [&](int piece) { return a.actions[(size_t)min(piece * kRelaySteps + (L.y & (kRelaySteps - 1)), nsteps - 1) * a.B + wm.envl]; };
  int act_next = action_of(0);
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // (the final state is stored after the barrier)
  __syncthreads();
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int i = 0; i < PR::P; ++i) arrived(p[i]);
  arrived(fz, er0.x, er0.y, er0.z, er0.w, er1.x, er1.y, act_next);
  EnvRec er;
  er.t = (int32_t)er0.y;
  er.n_changes = (int32_t)er0.z;
  er.episode = (int32_t)er0.w;
  er.key = (uint64_t)er1.x | ((uint64_t)er1.y << 32);
  er.pad_ = 0;
  int h = (int)(er0.x & 0xffu), w = (int)((er0.x >> 8) & 0xffu), py = (int)((er0.x >> 16) & 0xffu), px = (int)(er0.x >> 24);
  const bool random = a.pos_mode == kPosRandom;
  int max_steps = a.max_steps, max_changes = a.max_changes, autoreset = a.autoreset;
  asm volatile("" : "+s"(max_steps), "+s"(max_changes), "+s"(autoreset));
  int buf = 0, row_changes = 0;
  for (int piece = 0; piece < pieces; ++piece) {
    const int n = min(kRelaySteps, nsteps - piece * kRelaySteps);
    const int act_y = act_next;
    act_next = action_of(piece + 1);  // (wanted a piece later)
    const bool in_range_y = act_y >= 0 && act_y < PR::K;
    const uint64_t bad = __builtin_amdgcn_ballot_w64(wm.primary && L.y < n && !in_range_y);
    if (bad != 0 && L.lane == 0) atomicAdd(a.bad_actions, (unsigned long long)__popcll(bad));
    const uint32_t what_y = (uint32_t)(act_y & 7) << 16 | (in_range_y ? 1u << 19 : 0u);
    auto prepared = [&](int i) {  // lane y: step y, the next one being step i
      uint32_t v = what_y;
      if (random) {
        const uint64_t u = draw(er.key, 3, (uint32_t)(er.t + 1 + L.y - i));
        v |= (uint32_t)below((uint32_t)(u >> 32), h) | (uint32_t)below((uint32_t)u, w) << 8;
      }
      return (int)v;
    };
    int steps_y = prepared(0);
    uint32_t step_v = (uint32_t)L.gread_i(steps_y, 0);
    for (int i = 0; i < n; ++i) {
      const uint32_t v = step_v;
      step_v = (uint32_t)L.gread_i(steps_y, i + 1);
      const W cell = wm.valid && L.y == py ? (W)1 << px : (W)0;
      const int act = (int)((v >> 16) & 7u);
      int old_code = 0;
#pragma unroll
      for (int k = 0; k < PR::P; ++k) old_code |= (p[k] & cell) != 0 ? 1 << k : 0;
      const bool changed = cell != 0 && (v >> 19 & 1u) != 0 && (fz & cell) == 0 && act != old_code;  // in the row's lane
      if (changed) {
#pragma unroll
        for (int k = 0; k < PR::P; ++k) p[k] = (p[k] & ~cell) | ((act >> k) & 1 ? cell : (W)0);
      }
      er.t += 1;
      bool done = er.t >= max_steps;
      if (max_changes > 0) {
        er.n_changes += L.gany(changed) ? 1 : 0;
        done = done || er.n_changes >= max_changes;
      } else {
        row_changes += changed ? 1 : 0;  // (put together at the end)
      }
      const bool restart = wm.valid && done && autoreset != 0;
      int qy = (int)(v & 0xffu), qx = (int)((v >> 8) & 0xffu);
      if (!random) {
        qy = py;
        qx = px + 1;
        if (qx >= w) {
          qx = 0;
          qy += 1;
          if (qy >= h) qy = 0;
        }
      }
      uint2 r;
      r.x = (uint32_t)act | (uint32_t)old_code << 3 | (changed ? kTraceChanged : 0u) | (done ? kTraceDone : 0u) | (restart ? kTraceRestart : 0u);
      const uint32_t here = (uint32_t)py | (uint32_t)px << 8;
      const bool writer = wm.primary && L.y == py;
      if (wave_any<S>(restart)) {
        const KArgs& ra = cold_args<true>();
        W np[PR::P], nfz;
        int nh, nw, npy, npx;
        const uint64_t nkey = env_key(ra.seed, (uint64_t)wm.envl, (uint64_t)(er.episode + 1));
        begin_episode<S, PROBLEM, true, kDrawsAbreast<S, PROBLEM, false>>(ra, L, nkey, np, nfz, nh, nw, npy, npx, restart, wm.envl);
        if (restart) {
#pragma unroll
          for (int k = 0; k < PR::P; ++k) p[k] = np[k];
          fz = nfz;
          h = nh;
          w = nw;
          qy = npy;
          qx = npx;
          if (wm.primary) {
#pragma unroll
            for (int k = 0; k < PR::P; ++k) tables.rows[buf][wm.sl.slot][k][L.y] = np[k];
            tables.rows[buf][wm.sl.slot][PR::P][L.y] = nfz;
            if (L.y == 0) tables.hw[buf][wm.sl.slot] = nh | nw << 8;
          }
          er.key = nkey;
          er.episode += 1;
          er.t = 0;
          er.n_changes = 0;
          row_changes = 0;
        }
        steps_y = prepared(i + 1);
        step_v = (uint32_t)L.gread_i(steps_y, i + 1);
      }
      r.y = here | (uint32_t)qy << 16 | (uint32_t)qx << 24;
      if (writer) tables.trace[buf][i][wm.sl.slot] = r;
      py = qy;
      px = qx;
    }
    buf = buf == 2 ? 0 : buf + 1;
    relay_barrier();
  }
  relay_barrier();
  er.n_changes += L.gsum(row_changes);
  if (wm.primary) {
#pragma unroll
    for (int i = 0; i < PR::P; ++i) planes[(size_t)i * a.plane_stride + ridx] = p[i];
    frozen[ridx] = fz;
  }
  er.cell_frozen = L.gany(L.y == py && ((fz >> px) & 1)) ? 1u : 0u;
  if (wm.primary && L.y == 0) {
    er.h = (uint8_t)h;
    er.w = (uint8_t)w;
    er.py = (uint8_t)py;
    er.px = (uint8_t)px;
    a.env[wm.env] = er;
  }
}

// What searchers and observers have in common: their own copy of the levels, taken through the traced
// steps.
template <int S, int PROBLEM> struct RelayFollower {
  using W = typename RowWord<S>::T;
  using PR = Prob<PROBLEM>;
  W p[PR::P], fz, inside;
  int h, w;
  __device__ __forceinline__ void load(const KArgs& a, const Lanes<S>& L, const WaveMap<S>& wm) {
    const size_t ridx = (size_t)wm.envl * S + L.y;
#pragma unroll
    for (int i = 0; i < PR::P; ++i) p[i] = reinterpret_cast<const W*>(a.planes)[(size_t)i * a.plane_stride + ridx];
    fz = reinterpret_cast<const W*>(a.frozen)[ridx];
    const uint32_t hw = *reinterpret_cast<const uint32_t*>(a.env + wm.envl);
    h = (int)(hw & 0xffu);
    w = (int)((hw >> 8) & 0xffu);
  }
  __device__ __forceinline__ void loaded(const Lanes<S>& L) {
#pragma unroll
    for (int i = 0; i < PR::P; ++i) arrived(p[i]);
    arrived(fz, h, w);
    inside = inside_row<W>(L.y, h, w);
  }
  // (the lane of the row alone has a cell)
  __device__ __forceinline__ void edit(W cell, int act) {
#pragma unroll
    for (int i = 0; i < PR::P; ++i) p[i] = (p[i] & ~cell) | ((act >> i) & 1 ? cell : (W)0);
  }
  __device__ __forceinline__ void restart(const Lanes<S>& L, const RelayTables<S, PROBLEM>& tables, int buf, int level) {
#pragma unroll
    for (int i = 0; i < PR::P; ++i) p[i] = tables.rows[buf][level][i][L.y];
    fz = tables.rows[buf][level][PR::P][L.y];
    const int hw = tables.hw[buf][level];
    h = hw & 0xff;
    w = hw >> 8;
    inside = inside_row<W>(L.y, h, w);
  }
};

// A searcher.  The change of the region count and the paths depend on the level before and after the
// edit alone, and path values that an edit leaves as they are need not be known.  Binary problem: the
// component of the first walkable cell is kept until an edit touches it, at whoever's turn, and searched
// for again at the next own turn that needs it.
template <int S, int PROBLEM>
__device__ __forceinline__ void relay_searcher(const KArgs& a, const Lanes<S>& L, const WaveMap<S>& wm, int turn, int turn_mask,
                                               RelayTables<S, PROBLEM>& tables) {
  using W = typename RowWord<S>::T;
  using PR = Prob<PROBLEM>;
  RelayFollower<S, PROBLEM> f;
  f.load(a, L, wm);
  W comp = 0;
  if constexpr (PROBLEM == kBinary)
    comp = reinterpret_cast<const W*>(a.planes)[(size_t)PR::P * a.plane_stride + (size_t)wm.envl * S + L.y];
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  __builtin_amdgcn_sched_barrier(0);
  f.loaded(L);
  arrived(comp);
  bool comp_known = true;
  int mode = a.regions_mode;
  asm volatile("" : "+s"(mode));
  const int nsteps = a.rollout_steps, pieces = relay_pieces(nsteps);
  int buf = 0;
  relay_barrier();
  for (int piece = 0; piece < pieces; ++piece) {
    const int n = min(kRelaySteps, nsteps - piece * kRelaySteps), half = piece & 1;
    uint2 next = tables.trace[buf][0][wm.sl.slot];
    for (int i = 0; i < n; ++i) {
      const uint2 r = next;
      next = tables.trace[buf][min(i + 1, n - 1)][wm.sl.slot];
      const bool mine = ((piece * kRelaySteps + i) & turn_mask) == turn;
      const int act = (int)(r.x & 7u), py = (int)(r.y & 0xffu), px = (int)((r.y >> 8) & 0xffu);
      const bool changed = wm.valid && (r.x & kTraceChanged) != 0, restart = wm.valid && (r.x & kTraceRestart) != 0;
      const W cell = changed && L.y == py ? (W)1 << px : (W)0;
      f.edit(cell, act);
      if (mine) {
        Moved mv = {0, 0, 0, false};
        if (wave_any<S>(changed)) {
          mv = after_edit<S, PROBLEM>(mode == kRegionsRecount, L, f.p, f.inside, changed, (int)(r.x >> 3 & 7u), act, f.h, f.w, py, px, comp, comp_known);
          comp_known = comp_known || mv.searched;
        }
        if (wm.primary && L.y == 0)
          tables.found[half][i][wm.sl.slot] = make_uint2((mv.searched ? 1u : 0u) | (uint32_t)mv.regions << 16, (uint32_t)mv.path | (uint32_t)mv.enemy << 16);
      } else if constexpr (PROBLEM == kBinary) {
        if (wave_any<S>(changed && comp_known)) {
          const bool untouched = diameter_untouched<S>(L, comp, cell, L.dilate(cell), py, px, act != 1);
          comp_known = comp_known && (!changed || untouched);
        }
      }
      if (wave_any<S>(restart)) {
        if (restart) f.restart(L, tables, buf, wm.sl.slot);
        W ncomp = 0;
        if (mine) {
          int nm[PR::M];
          full_metrics<S, PROBLEM>(L, f.p, f.inside, restart, nm, ncomp);
          int v = 0;
#pragma unroll
          for (int k = 0; k < PR::M; ++k) v = L.y == k ? nm[k] : v;
          if (restart && wm.primary && L.y < kMaxMetrics) tables.metrics[half][wm.sl.slot][L.y] = v;
        }
        if (restart) {
          comp = ncomp;
          comp_known = mine;
        }
      }
    }
    buf = buf == 2 ? 0 : buf + 1;
    relay_barrier();
  }
  if constexpr (PROBLEM == kBinary) {  // the last turn's wavefront leaves the component behind
    if (((nsteps - 1) & turn_mask) == turn) {
      if (wave_any<S>(!comp_known)) {
        const W pass = comp_known ? (W)0 : (W)(f.inside & ~channel_row<PROBLEM, W>(f.p, f.inside, 1));
        W far, all;
        sweep<S>(L, first_cell<S>(L, pass), pass, far, all);
        comp = comp_known ? comp : all;
      }
      if (wm.primary) reinterpret_cast<W*>(a.planes)[(size_t)PR::P * a.plane_stride + (size_t)wm.envl * S + L.y] = comp;
    }
  }
}

// An observer.
template <int S, int PROBLEM>
__device__ __forceinline__ void relay_observer(KArgs a, const Lanes<S>& L, const WaveMap<S>& wm, int turn, int turn_mask,
                                               int level0, const RelayTables<S, PROBLEM>& tables) {
  using W = typename RowWord<S>::T;
  const int nsteps = a.rollout_steps, pieces = relay_pieces(nsteps);
  if (wm.env0 >= a.B) {  // the batch ends inside this workgroup: only the barriers are owed
    __syncthreads();
    for (int piece = 0; piece < pieces + 1; ++piece) relay_barrier();
    return;
  }
  RelayFollower<S, PROBLEM> f;
  f.load(a, L, wm);
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  __builtin_amdgcn_sched_barrier(0);
  f.loaded(L);
  // (each a register of its own: the compiler would otherwise hold on to the whole pieces of the argument
  // block they come in, and set stack space aside for those)
  asm volatile("" : "+s"(a.env_obs_bytes), "+s"(a.obs_packed), "+s"(a.obs_frozen_channel), "+s"(a.stream_obs));
  int slot = 0, buf = 0;
  relay_barrier();
  for (int piece = 0; piece < pieces; ++piece) {
    const int n = min(kRelaySteps, nsteps - piece * kRelaySteps);
    uint2 next = tables.trace[buf][0][level0 + wm.sl.slot];
    for (int i = 0; i < n; ++i) {
      const uint2 r = next;
      next = tables.trace[buf][min(i + 1, n - 1)][level0 + wm.sl.slot];
      const bool changed = wm.valid && (r.x & kTraceChanged) != 0, restart = wm.valid && (r.x & kTraceRestart) != 0;
      f.edit(changed && L.y == (int)(r.y & 0xffu) ? (W)1 << (r.y >> 8 & 0xffu) : (W)0, (int)(r.x & 7u));
      if (restart) f.restart(L, tables, buf, level0 + wm.sl.slot);
      if (((piece * kRelaySteps + i) & turn_mask) == turn) {
        // (the plan anew: kept from step to step it ties up scalar registers that this wavefront lacks)
        const ObsPlan pl = obs_plan(a, L.lane, wm.sl, a.obs + (size_t)slot * ((size_t)a.B * (size_t)a.env_obs_bytes), wm.env0, wm.nvalid);
        observe<S, PROBLEM, false, true>(a, L, wm, pl, f.p, f.fz, f.inside, (int)(r.y >> 16 & 0xffu), (int)(r.y >> 24));
      }
      slot = slot + 1 == a.obs_slots ? 0 : slot + 1;  // (step t writes slot t mod obs_slots)
    }
    buf = buf == 2 ? 0 : buf + 1;
    relay_barrier();
  }
}

// The adder.
template <int S, int PROBLEM>
__device__ __forceinline__ void relay_adder(const KArgs& a, const Lanes<S>& L, const WaveMap<S>& wm, const RelayTables<S, PROBLEM>& tables) {
  using PR = Prob<PROBLEM>;
  const int yi = L.y & (kMaxMetrics - 1);
  const size_t mrow = (size_t)wm.envl * kMaxMetrics;
  int m_l = a.metrics[mrow + yi];
  uint32_t tg_l = a.targets[mrow + yi];
  float w_l = __uint_as_float((a.targets - kMaxMetrics)[yi]);  // (the row in front of the ranges)
  int episode = a.env[wm.envl].episode;
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  __builtin_amdgcn_sched_barrier(0);
  arrived(m_l, tg_l, w_l, episode);
  const int nsteps = a.rollout_steps, pieces = relay_pieces(nsteps);
  bool targets_dirty = false;
  int buf = 0;
  relay_barrier();
  relay_barrier();
  for (int piece = 0; piece < pieces; ++piece) {
    const int n = min(kRelaySteps, nsteps - piece * kRelaySteps), half = piece & 1;
    uint2 next = tables.trace[buf][0][wm.sl.slot], next_found = tables.found[half][0][wm.sl.slot];
    for (int i = 0; i < n; ++i) {
      const uint2 r = next, fd = next_found;
      next = tables.trace[buf][min(i + 1, n - 1)][wm.sl.slot];
      next_found = tables.found[half][min(i + 1, n - 1)][wm.sl.slot];
      const bool changed = wm.valid && (r.x & kTraceChanged) != 0, searched = changed && (fd.x & 1u) != 0;
      const int act = (int)(r.x & 7u), old_code = (int)(r.x >> 3 & 7u), regions = (int)fd.x >> 16;
      const int k = yi - PR::CNT;
      int mn_l = m_l + (changed && act == k ? 1 : 0) - (changed && old_code == k ? 1 : 0);
      if (changed && yi == 0) mn_l = a.regions_mode == kRegionsRecount ? regions : m_l + regions;
      if (searched && yi == 1) mn_l = (int)(fd.y & 0xffffu);
      if (PROBLEM == kDungeon && searched && yi == 2) mn_l = (int)(fd.y >> 16);
      const float acc = reward_of<PR::M>(m_l, mn_l, tg_l, w_l);
      const size_t out = (size_t)(piece * kRelaySteps + i) * a.B + wm.env;
      if (wm.primary && L.y == PR::M - 1 && a.reward) a.reward[out] = changed ? acc : 0.0f;
      if (wm.primary && L.y == 0 && a.done) a.done[out] = (r.x & kTraceDone) != 0 ? 1 : 0;
      const bool restart = wm.valid && (r.x & kTraceRestart) != 0;
      if (wave_any<S>(restart)) {
        if (restart) mn_l = tables.metrics[half][wm.sl.slot][yi];
        const KArgs& ra = cold_args<true>();
        if (restart && ra.ctrl_mask != 0) {
          if ((ra.ctrl_mask >> yi) & 1u)
            tg_l = control_target(ra, env_key(ra.seed, (uint64_t)wm.envl, (uint64_t)(episode + 1)), yi);
          targets_dirty = true;
        }
        episode += restart ? 1 : 0;
      }
      m_l = mn_l;
    }
    buf = buf == 2 ? 0 : buf + 1;
    if (piece + 1 < pieces) relay_barrier();
  }
  if (wm.primary && L.y < PR::M) {
    a.metrics[(size_t)wm.env * kMaxMetrics + L.y] = m_l;
    if (targets_dirty) a.targets[(size_t)wm.env * kMaxMetrics + L.y] = tg_l;
  }
}

template <int S, int PROBLEM>
__global__ __launch_bounds__(640) void rollout_relay_kernel(KArgs a) {
  extern __shared__ __align__(16) uint32_t lds_all[];
  __shared__ RelayTables<S, PROBLEM> tables;
  Lanes<S> L;
  WaveMap<S> wm;
  const int wid = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int lg = a.envs_per_wave_log2 & 0xff, lgo = (a.envs_per_wave_log2 >> 8) & 0xff;
  const int searchers = 1 << ((a.envs_per_wave_log2 >> 24) & 0x7f);
  const int group = level_group_of_block<true>(a.by_die);
  if (wid >= 2 + searchers) {
    const int o = wid - 2 - searchers, share = o & ((1 << (lg - lgo)) - 1);
    wm.init(a, L, lds_all + o * a.obs_lds_words, (group << (lg - lgo)) + share, lgo);
    relay_observer<S, PROBLEM>(a, L, wm, o >> (lg - lgo), (1 << ((a.envs_per_wave_log2 >> 16) & 0xff)) - 1, share << lgo, tables);
    __builtin_amdgcn_endpgm();
  }
  wm.init(a, L, lds_all, group, lg);
  if (wid >= 2) {
    relay_searcher<S, PROBLEM>(a, L, wm, wid - 2, searchers - 1, tables);
    __builtin_amdgcn_endpgm();
  }
  if (wid == 1) {
    relay_adder<S, PROBLEM>(a, L, wm, tables);
    __builtin_amdgcn_endpgm();
  }
  relay_leader<S, PROBLEM>(a, L, wm, tables);
}

// The body of the two kernels below.  On entry `a` holds what a step needs to request its loads
// (the six state pointers, B, plane_stride, envs_per_wave_log2, use_frozen); a rollout has all of it.
// PIN = false is the same code for contexts none of whose levels has a pinpoint cell
// (use_frozen == 0; single steps only): what looks pinpoints up is left out, which frees enough
// registers for one more wavefront per SIMD on 64-row levels (all 8192 wavefronts of the 64x64
// maze at a batch of 8192 resident at once, -2.3 % per step; 32x32 dungeon -2.8 %).  WIDTH: which
// form of the observation code a single step carries (see observe); a rollout carries both.
// (last_span: the span of a rollout that this workgroup runs is its last one)
template <int S, int PROBLEM, int MODE, bool PIN, int WIDTH>
__device__ __forceinline__ void step_body(KArgs& a, [[maybe_unused]] bool last_span = false) {
  using W = typename RowWord<S>::T;
  using PR = Prob<PROBLEM>;
  constexpr bool ROLL = MODE >= kModeRollout, SPAN = MODE == kModeSpan;
  constexpr bool TRIPS = S == 32 && (!ROLL || SPAN);  // (see flood_to_end)
  constexpr bool SPLIT = MODE != kModeStep && MODE != kModeRollout;
  // Whether what a rollout needs rarely or at its end is looked up in the argument block again instead of
  // being kept in scalar registers, of which the step loop has too few: it spills them to vector
  // registers and reads them back in every step.  Us a step without / with: 8192 32x32 maze levels 4.08 / 3.68,
  // 64x64 dungeons 7.10 / 6.92, 65 536 32x32 binary levels 20.9 / 20.5, 8192 16x16 dungeons without
  // observations 2.10 / 2.04.  Not for split rollouts of 16-row levels (8192 binary levels 4.85 / 4.91, 2048 maze
  // levels 2.42 / 2.49) and, one wavefront a level, 64-row binary and maze levels (12 288 maze levels 12.7 / 12.9).
  // (A span's state comes from one place and goes to another: the block holds the latter.)
  constexpr bool LOOK_UP = SPAN || (ROLL && (SPLIT ? S > 16 : S < 64 || PROBLEM == kDungeon));
  extern __shared__ __align__(16) uint32_t lds_all[];
  Lanes<S> L;
  WaveMap<S> wm;
  wm.init(a, L, lds_all, level_group_of_block<ROLL>(ROLL ? a.by_die : 0), a.envs_per_wave_log2 & 0xff);
  // SPLIT: the workgroup is two wavefronts on the same levels; wavefront 0 does the metrics, the
  // reward and the state stores (the code below, without its observation parts), wavefront 1 the
  // observation; both load the same (old) state
  if constexpr (SPLIT) {
    // wavefront 0 of the workgroup computes the metrics of 1 << lg levels; each further wavefront
    // writes the observations of 1 << lgo of them (a copy of the level in every spare lane group)
    const int wid = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    if (wid != 0) {
      const int lg = a.envs_per_wave_log2 & 0xff, lgo = (a.envs_per_wave_log2 >> 8) & 0xff;
      // (wavefronts 1 .. n of a rollout share out the levels of the group, the next n take the
      // same levels at the next turn, and so on)
      const int share = ROLL ? (wid - 1) & ((1 << (lg - lgo)) - 1) : wid - 1;
      wm.init(a, L, nullptr, (level_group_of_block<ROLL>(ROLL ? a.by_die : 0) << (lg - lgo)) + share, lgo);
      if constexpr (ROLL) {
        wm.lds = lds_all + (wid - 1) * a.obs_lds_words;
        const int turn_mask = (1 << ((a.envs_per_wave_log2 >> 16) & 0xff)) - 1;
        obs_wave_rollout<S, PROBLEM, MODE == kModeRolloutTurns>(a, L, wm, (wid - 1) >> (lg - lgo), turn_mask);
      } else {
        obs_wave_step<S, PROBLEM, PIN, WIDTH>(a, L, wm, lds_all, wid);
      }
      __builtin_amdgcn_endpgm();  // (not a return: the two paths must not meet again, or the
                                  // compiler makes this one wait for the other one's loads)
    }
  }
  const bool valid = wm.valid;
  W* planes = reinterpret_cast<W*>(a.planes);
  W* frozen = reinterpret_cast<W*>(a.frozen);
  const size_t ridx = (size_t)wm.envl * S + L.y;

  // ---- load: everything the step needs is requested up front (one memory round trip)
  W p[PR::P];
#pragma unroll
  for (int i = 0; i < PR::P; ++i) p[i] = planes[(size_t)i * a.plane_stride + ridx];
  W fz = 0;  // pinpoint rows: resident only in a rollout; a single step keeps a flag with the cell
  if (ROLL || (PIN && (a.use_frozen & 2))) fz = frozen[ridx];
  // binary problem: the component of the first walkable cell, which is all that the diameter
  // estimate depends on; an edit elsewhere needs no sweep (see diameter_untouched)
  W comp = 0;
  bool comp_dirty = false;
  if constexpr (PROBLEM == kBinary && !SPAN) comp = planes[(size_t)PR::P * a.plane_stride + ridx];
  const uint4* erp = reinterpret_cast<const uint4*>(a.env + wm.envl);
  const uint4 er0 = erp[0], er1 = erp[1];  // unpacked below, after all loads are under way
  int act = a.actions[wm.envl];  // (lanes without a level of their own read a neighbour's and ignore it)
  // The metric vector, its target ranges and the reward weights are kept one entry per lane
  // (lane y of a group holds entry y): what an edit does to them - one tile count up, one down, up
  // to three flood results replaced, one loss difference per metric - is then a handful of
  // instructions for the whole vector instead of a handful per metric.  Only the region count is
  // also needed by every lane (the incremental update starts from it).
  const int yi = L.y & (kMaxMetrics - 1);
  const size_t mrow = (size_t)wm.envl * kMaxMetrics;
  int m_l = 0, regions_now = 0;  // (a span has them from scratch, below)
  if constexpr (!SPAN) m_l = a.metrics[mrow + yi];
  uint32_t tg_l = a.targets[mrow + yi];
  if constexpr (!SPAN) regions_now = a.metrics[mrow];
  const float w_l = __uint_as_float(((SPAN ? cold_args<true>().targets : a.targets) - kMaxMetrics)[yi]);  // (the row in front of the ranges)
  // every load above is issued before anything below waits for one of them; now the rest of the
  // arguments is fetched, in their shadow
  __builtin_amdgcn_sched_barrier(0);
  if constexpr (!ROLL) fill_rest_of_args(a);
  // the observation wavefront has received the old state before this wavefront goes on to store
  // the new one (this wavefront passes the barrier with its own loads still in flight)
  if constexpr (SPLIT) {
    __syncthreads();
    __builtin_amdgcn_sched_barrier(0);
  }
  // a single step stages one observation: where it goes is worked out, and its LDS words are
  // cleared, in the shadow of the loads
  ObsPlan pl;
  if constexpr (MODE == kModeStep) {
    pl = obs_plan(a, L.lane, wm.sl, a.obs, wm.env0, wm.nvalid);
    obs_plan_pin(pl);
    if (a.obs != nullptr) obs_clear(wm.lds, L.lane, pl);
    __builtin_amdgcn_sched_barrier(0);
  }
  EnvRec er;
  er.t = (int32_t)er0.y;
  er.n_changes = (int32_t)er0.z;
  er.episode = (int32_t)er0.w;
  er.key = (uint64_t)er1.x | ((uint64_t)er1.y << 32);
  er.cell_frozen = er1.z;
  er.pad_ = 0;
  int h = (int)(er0.x & 0xffu), w = (int)((er0.x >> 8) & 0xffu), py = (int)((er0.x >> 16) & 0xffu), px = (int)(er0.x >> 24);
  W inside = inside_row<W>(L.y, h, w);
  bool planes_dirty = false, fz_dirty = false;  // ROLL: what has to be written back at the end
  bool metrics_dirty = false, targets_dirty = false;
  if constexpr (SPAN) {  // nobody has followed the metrics as far as here
    int m[PR::M];
    full_metrics<S, PROBLEM, TRIPS>(L, p, inside, valid, m, comp);
#pragma unroll
    for (int i = 0; i < PR::M; ++i)
      if (yi == i) m_l = m[i];
    regions_now = m[0];
  }
  W next_fz_row = 0;
  uint32_t next_cell_frozen = 0;

  const int nsteps = ROLL ? a.rollout_steps : 1;
  // (a rollout that writes its own observations: the plan of slot 0 serves every slot whose
  // address differs from it by a multiple of 16 bytes, see obs_wave_rollout)
  [[maybe_unused]] int slot = 0;
  [[maybe_unused]] size_t slot_off = 0;
  [[maybe_unused]] size_t slot_bytes = 0;
  [[maybe_unused]] bool fixed_plan = false;
  [[maybe_unused]] uint8_t* base0 = nullptr;
  if constexpr (ROLL && !SPLIT) {
    if (a.obs != nullptr) {
      slot_bytes = (size_t)a.B * (size_t)a.env_obs_bytes;
      fixed_plan = (slot_bytes & 15u) == 0;
      pl = obs_plan(a, L.lane, wm.sl, a.obs, wm.env0, wm.nvalid);
      base0 = pl.base;
    }
  }
  for (int step = 0; step < nsteps; ++step) {
    // the next step's action is requested now and used one iteration later
    int act_next = -1;
    if constexpr (ROLL) {
      if (step + 1 < nsteps) act_next = a.actions[(size_t)(step + 1) * a.B + wm.envl];
    }
    uint8_t* obs = a.obs;
    if constexpr (ROLL && !SPLIT) {
      if (obs != nullptr) {
        if (fixed_plan) pl.base = base0 + slot_off;
        else pl = obs_plan(a, L.lane, wm.sl, obs + slot_off, wm.env0, wm.nvalid);
        slot = slot + 1 == a.obs_slots ? 0 : slot + 1;  // (step t writes slot t mod obs_slots)
        slot_off = slot == 0 ? 0 : slot_off + slot_bytes;
      }
    }

    // ---- edit (Methods / Training: the agent may change the tile it stands on)
    const bool at_row = L.y == py;
    int old_code = 0;
#pragma unroll
    for (int i = 0; i < PR::P; ++i) old_code |= (L.gany(at_row && ((p[i] >> px) & 1)) ? 1 : 0) << i;
    bool is_frozen;
    if constexpr (ROLL) is_frozen = L.gany(at_row && ((fz >> px) & 1));
    else is_frozen = PIN && er.cell_frozen != 0;
    const bool in_range = act >= 0 && act < PR::K;
    const bool changed = valid && in_range && !is_frozen && act != old_code;
    if (__builtin_amdgcn_ballot_w64((uint32_t)act >= (uint32_t)PR::K) != 0) {  // rare: count them
      const uint64_t bad = __builtin_amdgcn_ballot_w64(wm.primary && !in_range && L.y == 0);
      if (bad != 0 && L.lane == 0) atomicAdd(LOOK_UP ? cold_args<ROLL>().bad_actions : a.bad_actions, (unsigned long long)__popcll(bad));
    }
    if (changed && at_row) {
#pragma unroll
      for (int i = 0; i < PR::P; ++i) {
        p[i] = (p[i] & ~((W)1 << px)) | ((W)((act >> i) & 1) << px);
        if constexpr (!ROLL) {
          if (wm.primary) planes[(size_t)i * a.plane_stride + ridx] = p[i];
        }
      }
      planes_dirty = true;
    }
    metrics_dirty = metrics_dirty || changed;
    // ---- counters, done flag and the agent's next cell need nothing but the edit
    er.t += 1;
    er.n_changes += changed ? 1 : 0;
    const bool done = (er.t >= a.max_steps) || (a.max_changes > 0 && er.n_changes >= a.max_changes);
    const bool restart = valid && done && a.autoreset != 0;
    int qy = py, qx = px;
    if (a.pos_mode == kPosScan) {
      qx += 1;
      if (qx >= w) {
        qx = 0;
        qy += 1;
        if (qy >= h) qy = 0;
      }
    } else {
      uint64_t u = draw(er.key, 3, (uint32_t)er.t);
      qy = below((uint32_t)(u >> 32), h);
      qx = below((uint32_t)u, w);
    }
    // pinpoint flag of the cell the next step will edit (one word, off the critical path)
    if constexpr (!ROLL) {
      if constexpr (PIN) {
        if (a.use_frozen) next_fz_row = frozen[(size_t)wm.envl * S + qy];
      }
    }
    // ---- observation around the new position.  It needs only the edited map and the new cell,
    // so it is issued before the metrics and its stores drain while the floods run; a wavefront
    // in which some level restarts writes it last, from the new episode's level.  (Letting odd
    // wavefronts flood first and store later was measured and does not pay.)
    const bool any_restart = wave_any<S>(restart);
    const bool obs_late = any_restart;
    if constexpr (!SPLIT) {
      if (obs != nullptr && !obs_late) observe<S, PROBLEM, !ROLL, false, WIDTH>(a, L, wm, pl, p, fz, inside, qy, qx);
    }

    // ---- metrics, only where the edit modified the map (Methods / Task)
    int mn_l = m_l;               // this lane's entry of the new metric vector
    int regions_new = regions_now;
    float reward = 0.0f;          // (ends up in lane M-1 of the group)
    if (wave_any<S>(changed)) {
      const W in = changed ? inside : (W)0;  // unchanged levels look empty: their loops end at once
      const W wall = channel_row<PROBLEM, W>(p, in, 1);
      const W pass = in & ~wall;
      // tile counts: one cell moved from one tile type to another
      {
        const int k = yi - PR::CNT;  // the tile type whose count this lane keeps, if any
        mn_l += (changed && act == k ? 1 : 0) - (changed && old_code == k ? 1 : 0);
      }
      const bool was_pass = old_code != 1, now_pass = act != 1;
      // regions
      if (a.regions_mode == kRegionsRecount) {
        int rc = regions_full<S>(L, pass, in, true);
        if (changed) regions_new = rc;
      } else {
        const bool flip = changed && was_pass != now_pass;
        if (wave_any<S>(flip)) {
          const W cell = (flip && at_row) ? (W)1 << px : (W)0;
          int k;
          if constexpr ((S == 16 || (S == 32 && ROLL)) && PROBLEM == kBinary) {  // (see neighbour_components)
            const W passw = flip ? (W)(pass & ~cell) : (W)0;
            k = neighbour_components<S>(L, (L.dilate(cell) & ~cell) & passw, passw);
          } else {
            k = components_around<S>(L, flip ? (W)(pass & ~cell) : (W)0, inside, cell, h, w, py, px);
          }
          if (flip) regions_new = regions_now + (now_pass ? 1 - k : k - 1);
        }
      }
      if (yi == 0) mn_l = regions_new;
      // paths
      if constexpr (PROBLEM == kBinary) {
        // (every modifying edit of a binary level flips the walkability of its cell)
        const W cell = (changed && at_row) ? (W)1 << px : (W)0;
        const bool need = changed && !diameter_untouched<S>(L, comp, cell, L.dilate(cell), py, px, now_pass);
        if (wave_any<S>(need)) {
          W ncomp;
          int dm = two_sweep_diameter<S, TRIPS>(L, need ? pass : (W)0, ncomp);
          if (need) {
            comp = ncomp;
            comp_dirty = true;
            if (yi == 1) mn_l = dm;
            if constexpr (!ROLL) {
              if (wm.primary) planes[(size_t)PR::P * a.plane_stride + ridx] = ncomp;
            }
          }
        }
      } else if constexpr (PROBLEM == kMaze) {
        W r;
        int dd = nearest<S>(L, channel_row<PROBLEM, W>(p, in, 2), channel_row<PROBLEM, W>(p, in, 3), pass, r);
        if (changed && yi == 1) mn_l = dd < 0 ? 0 : dd;
      } else {
        // swapping empty and chest changes neither the graph nor any source or target set
        const bool plain = (old_code == 0 || old_code == 6) && (act == 0 || act == 6);
        const bool need = changed && !plain;
        if (wave_any<S>(need)) {
          const W inn = need ? in : (W)0;
          const W passn = need ? pass : (W)0;
          W k1, r;
          int d1, de;
          nearest_two<S>(L, channel_row<PROBLEM, W>(p, inn, 2), channel_row<PROBLEM, W>(p, inn, 3),
                         channel_row<PROBLEM, W>(p, inn, 5), passn, d1, k1, de);
          int d2 = nearest<S>(L, k1, channel_row<PROBLEM, W>(p, inn, 4), passn, r);
          if (need && yi == 1) mn_l = (d1 >= 0 && d2 >= 0) ? d1 + d2 : 0;
          if (need && yi == 2) mn_l = de < 0 ? 0 : de;
        }
      }
      const float sum = reward_of<PR::M>(m_l, mn_l, tg_l, w_l);
      if (changed) reward = sum;
    }
    // ---- auto-reset: fresh seeded episode for the finished levels; the others keep their registers
    if (any_restart) {
      const KArgs& ra = cold_args<ROLL>();
      W np[PR::P], nfz;
      int nh, nw, npy, npx;
      uint64_t nkey = env_key(ra.seed, (uint64_t)wm.envl, (uint64_t)(er.episode + 1));
      begin_episode<S, PROBLEM, true, kDrawsAbreast<S, PROBLEM, ROLL>>(ra, L, nkey, np, nfz, nh, nw, npy, npx, restart, wm.envl);
      W ninside = inside_row<W>(L.y, nh, nw);
      int nm[PR::M];
      W ncomp;
      full_metrics<S, PROBLEM, TRIPS>(L, np, ninside, restart, nm, ncomp);
      if (restart) {
#pragma unroll
        for (int i = 0; i < PR::P; ++i) {
          p[i] = np[i];
          if constexpr (!ROLL) {
            if (wm.primary) planes[(size_t)i * a.plane_stride + ridx] = np[i];
          }
        }
        if constexpr (PROBLEM == kBinary) {
          comp = ncomp;
          comp_dirty = true;
          if constexpr (!ROLL) {
            if (wm.primary) planes[(size_t)PR::P * a.plane_stride + ridx] = ncomp;
          }
        }
        fz = nfz;
        if constexpr (!ROLL && PIN) {  // (without pinpoints the stored rows are zero and stay zero)
          if (wm.primary) frozen[ridx] = nfz;
          next_fz_row = L.gread(nfz, npy);
        }
        planes_dirty = true;
        fz_dirty = true;
        metrics_dirty = true;
        if (ra.ctrl_mask != 0) {
          if ((ra.ctrl_mask >> yi) & 1u) tg_l = control_target(ra, nkey, yi);
          targets_dirty = true;
        }
#pragma unroll
        for (int i = 0; i < PR::M; ++i)
          if (yi == i) mn_l = nm[i];
        regions_new = nm[0];
        inside = ninside;
        h = nh;
        w = nw;
        qy = npy;
        qx = npx;
        er.key = nkey;
        er.episode += 1;
        er.t = 0;
        er.n_changes = 0;
      }
    }

    // ---- per-step outputs
    // (a single step takes the pinpoint flag of the next cell out of its loaded row here, before
    // the stores below are issued: waiting for that load later would wait for these stores too)
    if constexpr (!ROLL && PIN) {
      if (a.use_frozen) {  // (a branch, so that contexts without pinpoints skip the wait as well)
        next_cell_frozen = (uint32_t)((next_fz_row >> qx) & 1);
        asm volatile("" : "+v"(next_cell_frozen));
      }
    }
    if (wm.primary && L.y == PR::M - 1) {
      if (a.reward) a.reward[(size_t)step * a.B + wm.env] = reward;
    }
    if (wm.primary && L.y == 0) {
      if (a.done) a.done[(size_t)step * a.B + wm.env] = done ? 1 : 0;
    }
    if constexpr (!SPLIT) {
      if (obs != nullptr && obs_late) observe<S, PROBLEM, !ROLL, false, WIDTH>(a, L, wm, pl, p, fz, inside, qy, qx);
    }

    // ---- the new state becomes the current one
    py = qy;
    px = qx;
    m_l = mn_l;
    regions_now = regions_new;
    act = act_next;
  }

  // ---- store the level's scalars (and, after a rollout, everything that changed)
  if constexpr (SPAN) {  // (all but the metrics span_starts_kernel has stored)
    if (last_span && wm.primary) {
      const KArgs& to = cold_args<true>();
      if constexpr (PROBLEM == kBinary) reinterpret_cast<W*>(to.planes)[(size_t)PR::P * to.plane_stride + ridx] = comp;
      if (L.y < PR::M) to.metrics[(size_t)wm.env * kMaxMetrics + L.y] = m_l;
    }
    __builtin_amdgcn_endpgm();
  }
  const KArgs& fin = [&]() -> const KArgs& {
    if constexpr (LOOK_UP) return cold_args<ROLL>();
    else return a;
  }();
  if constexpr (ROLL) {
    planes = reinterpret_cast<W*>(fin.planes);
    if (wm.primary) {
      if (planes_dirty) {
#pragma unroll
        for (int i = 0; i < PR::P; ++i) planes[(size_t)i * fin.plane_stride + ridx] = p[i];
      }
      if (fz_dirty) reinterpret_cast<W*>(fin.frozen)[ridx] = fz;
      if constexpr (PROBLEM == kBinary) {
        if (comp_dirty) planes[(size_t)PR::P * fin.plane_stride + ridx] = comp;
      }
    }
    next_fz_row = L.gread(fz, py);
  }
  if (wm.primary && L.y == 0) {
    er.h = (uint8_t)h;
    er.w = (uint8_t)w;
    er.py = (uint8_t)py;
    er.px = (uint8_t)px;
    er.cell_frozen = ROLL ? (uint32_t)((next_fz_row >> px) & 1) : next_cell_frozen;
    fin.env[wm.env] = er;
  }
  if (wm.primary && L.y < PR::M) {
    if (metrics_dirty) fin.metrics[(size_t)wm.env * kMaxMetrics + L.y] = m_l;
    if (targets_dirty) fin.targets[(size_t)wm.env * kMaxMetrics + L.y] = tg_l;
  }
  if constexpr (SPLIT) __builtin_amdgcn_endpgm();  // see the observation wavefront's exit above
}

// One environment step of every level (pcgrl_step).  What a step needs to request its loads -- the
// six state pointers, the batch, the plane stride and the wave shape -- comes as leading scalar
// arguments of 14 dwords, which the library is compiled to have preloaded into scalar registers
// when a wavefront is launched (where the firmware cannot do that, the compiler's own prologue
// loads them): a wavefront then computes its addresses and issues its loads at once, instead of
// first waiting for a fetch of its argument block through caches that every launch starts with
// empty (64x64 maze at a batch of 8192: 16.3 -> 15.8 us per step).  The rest of the configuration
// follows as the block `rest`, which only fixes where that block lies among the arguments: it is
// read through fill_rest_of_args() once the loads are under way.
//   shape: batch | levels per wavefront (log2) << 25 | the same for an observation wavefront << 27
//          | use_frozen << 29
//
// One more thing the kernel has to see to itself: on the MI355X a 64-bit vector shift whose shift
// amount sits in the highest register of the wavefront's allocation (registers come in blocks of
// eight) returns wrong results in some lanes once several wavefronts share a SIMD, and the
// compiler does not avoid it on this target.  The build looks for such shifts in the assembly it
// produces and fails on a finding (build.py); a kernel it names is listed in kPadRegistersAbove
// with its allocation, and then claims one register of the next block, which it never uses.
template <int S, int PROBLEM, int MODE, bool PIN, bool WIDE> constexpr int kPadRegistersAbove = 0;
template <> constexpr int kPadRegistersAbove<64, kMaze, kModeStep, true, true> = 64;
// Makes the kernel's allocation reach past register N - 1 (a clobber the code never touches).
template <int N> __device__ __forceinline__ void claim_register_above() {
  static_assert(N == 0 || (N % 8 == 0 && N >= 40 && N <= 104), "an allocation is a multiple of eight registers");
  if constexpr (N == 40) asm volatile("" ::: "v40");
  if constexpr (N == 48) asm volatile("" ::: "v48");
  if constexpr (N == 56) asm volatile("" ::: "v56");
  if constexpr (N == 64) asm volatile("" ::: "v64");
  if constexpr (N == 72) asm volatile("" ::: "v72");
  if constexpr (N == 80) asm volatile("" ::: "v80");
  if constexpr (N == 88) asm volatile("" ::: "v88");
  if constexpr (N == 96) asm volatile("" ::: "v96");
  if constexpr (N == 104) asm volatile("" ::: "v104");
}
template <int S, int PROBLEM, int MODE, bool PIN, bool WIDE>
__global__ __launch_bounds__(MODE == kModeSplit ? 320 : 64) void step_kernel(
    void* planes_, void* frozen_, EnvRec* env_, int32_t* metrics_, uint32_t* targets_, const int32_t* actions_,
    uint32_t shape, int32_t plane_stride_, KArgs rest) {
  static_assert(MODE == kModeStep || MODE == kModeSplit, "single steps only");
  static_assert(alignof(KArgs) == 8 && 6 * sizeof(void*) + 8 == kStepArgsOffset, "cold_args() assumes this layout");
  (void)rest;
  KArgs a;
  a.planes = planes_;
  a.frozen = frozen_;
  a.env = env_;
  a.metrics = metrics_;
  a.targets = targets_;
  a.actions = actions_;
  a.B = (int32_t)(shape & 0x1ffffffu);
  a.plane_stride = plane_stride_;
  a.envs_per_wave_log2 = (int32_t)(((shape >> 25) & 3u) | (((shape >> 27) & 3u) << 8));
  a.use_frozen = (int32_t)((shape >> 29) & 3u);
  claim_register_above<kPadRegistersAbove<S, PROBLEM, MODE, PIN, WIDE>>();
  step_body<S, PROBLEM, MODE, PIN, WIDE ? kWidthWide : kWidthNarrow>(a);
}

// `rollout_steps` consecutive steps per launch (pcgrl_rollout), during which the levels never
// leave the registers: per step only the action is read and the observation, reward and done
// flag are written.  A launch per hundred steps has nothing to gain from preloaded arguments.
template <int S, int PROBLEM, int MODE>
__global__ __launch_bounds__(MODE == kModeRollout ? 64 : 320) void rollout_kernel(KArgs a) {
  static_assert(MODE >= kModeRollout, "rollouts only");
  step_body<S, PROBLEM, MODE, true, kWidthAny>(a);
}

// ---- Spans: a rollout of a small batch, cut up along its steps.
// A small batch leaves most of the machine idle while each of its levels goes through one dependent chain
// per step.  What the levels go through does not depend on the metrics, and costs next to nothing beside
// them, so one wavefront a level runs ahead through all the steps and writes down what the level looks like
// at the start of every span of `steps` steps; all spans of all levels are then taken through their steps
// at the same time, each by wavefronts of its own, which begin with the metrics from scratch.
// When, and into how many spans, csrc/pcgrl_spans.h says.  256 steps of 64 16x16 binary levels 150 -> 29.8 us (the
// relay before), 32 steps of 512 16x16 maze levels 32 -> 21, of 1024 32x32 dungeon levels 56 -> 44.
struct SpanArgs {
  void* planes;       // word [P][plane_stride], index (span * B + env) * S + y
  void* frozen;       // word [plane_stride]
  EnvRec* env;        // [spans * B]
  uint32_t* targets;  // [spans * B][16]
  int32_t plane_stride;
  int32_t spans, steps;  // spans of a rollout, and steps of a span (the last one may have fewer)
};

// The states at the starts of all spans, and the state after the rollout, all but its metrics.
// Lane i follows step i of the next 64: where the agent goes is one hash a lane, the tile it finds is that
// of the latest earlier step of the 64 on the same cell (few share one: `who` names one lane of a cell, and
// only those that do not find themselves there look at each other), and an edit is the exclusive or of the
// tile's code before and after, so that the edits of any run of steps go into the bit-planes in LDS at once,
// in any order.  A step that ends an episode ends the 64 steps early: what later ones did to the level is
// of no consequence, the new level takes its place.
// Bound by latency: 256 steps of 64 16x16 binary levels, 64 spans, 10.0 us, 32 steps of 64 64x64 maze levels 5.4, of which
// 3 are the launch, its loads and its stores.  The spans are shared out over kSpanStartWaves wavefronts, which all follow all
// steps (with one of them 9.8 us; each span is some 400 clocks of reading back and storing).
constexpr int kSpanStartWaves = 4;
template <int S, int PROBLEM>
__global__ __launch_bounds__(64 * kSpanStartWaves) void span_starts_kernel(KArgs a, SpanArgs sp) {
  using W = typename RowWord<S>::T;
  using PR = Prob<PROBLEM>;
  constexpr int kWords = sizeof(W) / 4;
  struct Tables {
    uint32_t rows[PR::P][kWords][S];  // the level's bit-planes
    uint32_t pins[kWords][S];         // its pinpoints
    uint8_t who[S * S];
  };
  __shared__ Tables tables[kSpanStartWaves];
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  auto& rows = tables[wave].rows;
  auto& pins = tables[wave].pins;
  auto& who = tables[wave].who;
  Lanes<S> L;
  WaveMap<S> wm;
  wm.init(a, L, nullptr, (int)blockIdx.x, 0);
  const int env = wm.env, lane = L.lane, n_steps = a.rollout_steps;
  const bool primary = wm.primary;
  const size_t ridx = (size_t)env * S + L.y;
  W p[PR::P];
#pragma unroll
  for (int k = 0; k < PR::P; ++k) p[k] = reinterpret_cast<const W*>(a.planes)[(size_t)k * a.plane_stride + ridx];
  W fz = reinterpret_cast<const W*>(a.frozen)[ridx];
  const uint4* erp = reinterpret_cast<const uint4*>(a.env + env);
  const uint4 er0 = erp[0], er1 = erp[1];
  const int yi = L.y & (kMaxMetrics - 1);
  uint32_t tg = a.targets[(size_t)env * kMaxMetrics + yi];
  bool targets_moved = false;
  auto action_at = [&](int step) { return a.actions[(size_t)min(step + lane, n_steps - 1) * a.B + env]; };
  int act_next = action_at(0);
  // (every wavefront has the old state before one of them stores the new one)
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  __builtin_amdgcn_sched_barrier(0);
  int h = (int)(er0.x & 0xffu), w = (int)((er0.x >> 8) & 0xffu), py = (int)((er0.x >> 16) & 0xffu), px = (int)(er0.x >> 24);
  int t = (int)er0.y, n_changes = (int)er0.z, episode = (int)er0.w;
  uint64_t key = (uint64_t)er1.x | ((uint64_t)er1.y << 32);
  // (a span's record leaves the pinpoint flag of the agent's cell out: a rollout looks at the rows)
  auto store_env = [&](EnvRec* to, uint32_t at, int t_, int n_changes_, uint32_t cell_frozen) {
    if (lane == 0) {
      uint4* r = reinterpret_cast<uint4*>(to);
      r[0] = make_uint4((uint32_t)h | (uint32_t)w << 8 | at << 16, (uint32_t)t_, (uint32_t)n_changes_, (uint32_t)episode);
      r[1] = make_uint4((uint32_t)key, (uint32_t)(key >> 32), cell_frozen, 0u);
    }
  };
  auto store_span = [&](int span, uint32_t at, int t_, int n_changes_) {
    const size_t i = (size_t)span * a.B + env, row = i * S + L.y;
    if (primary) {
#pragma unroll
      for (int k = 0; k < PR::P; ++k) reinterpret_cast<W*>(sp.planes)[(size_t)k * sp.plane_stride + row] = p[k];
      reinterpret_cast<W*>(sp.frozen)[row] = fz;
      if (L.y < PR::M) sp.targets[i * kMaxMetrics + L.y] = tg;
    }
    store_env(sp.env + i, at, t_, n_changes_, 0u);
  };
  auto level_to_lds = [&]() {
    if (primary) {
#pragma unroll
      for (int j = 0; j < kWords; ++j) {
#pragma unroll
        for (int k = 0; k < PR::P; ++k) rows[k][j][L.y] = (uint32_t)((uint64_t)p[k] >> (32 * j));
        pins[j][L.y] = (uint32_t)((uint64_t)fz >> (32 * j));
      }
    }
    lds_sync();
  };
  auto level_from_lds = [&]() {
    lds_sync();
#pragma unroll
    for (int k = 0; k < PR::P; ++k) {
      uint64_t v = rows[k][0][L.y];
      if constexpr (kWords == 2) v |= (uint64_t)rows[k][1][L.y] << 32;
      p[k] = (W)v;
    }
  };
  uint32_t at = (uint32_t)py | (uint32_t)px << 8;  // the agent's cell
  if (wave == 0) store_span(0, at, t, n_changes);
  level_to_lds();
  int span = wave == 0 ? kSpanStartWaves : wave;  // the next one for this wavefront to store
  for (int done_steps = 0; done_steps < n_steps;) {
    const int n = min(64, n_steps - done_steps);
    const int act = act_next;
    act_next = action_at(done_steps + n);
    // the agent's cell after this lane's step, and before it
    uint32_t after;
    if (a.pos_mode == kPosRandom) {
      const uint64_t u = draw(key, 3, (uint32_t)(t + 1 + lane));
      after = (uint32_t)below((uint32_t)(u >> 32), h) | (uint32_t)below((uint32_t)u, w) << 8;
    } else {
      const uint32_t j = ((at & 0xffu) * (uint32_t)w + (at >> 8) + (uint32_t)lane + 1u) % (uint32_t)(h * w);
      after = j / (uint32_t)w | (j % (uint32_t)w) << 8;
    }
    uint32_t before = dpp_zero_fill<kWaveShr1>(after);
    if (lane == 0) before = at;
    lds_sync();
    const int y = (int)(before & 0xffu), x = (int)(before >> 8), word = x >> 5, cell = y * S + x;
    int old = 0;
#pragma unroll
    for (int k = 0; k < PR::P; ++k) old |= (int)((rows[k][word][y] >> (x & 31)) & 1u) << k;
    const bool pinned = ((pins[word][y] >> (x & 31)) & 1u) != 0;
    const bool may_write = lane < n && act >= 0 && act < PR::K && !pinned;
    // the tile the step finds: that of the latest earlier one on the same cell, if there is one
    if (may_write) who[cell] = (uint8_t)lane;
    lds_sync();
    uint64_t clash = __builtin_amdgcn_ballot_w64(may_write && who[cell] != (uint8_t)lane);
    if (clash != 0) {
      uint64_t same = 0;
      do {  // (once for every cell that several steps share)
        const int c = __builtin_amdgcn_readlane(cell, (int)__builtin_ctzll(clash));
        const bool here = may_write && cell == c;
        const uint64_t all = __builtin_amdgcn_ballot_w64(here);
        if (here) same = all;
        clash &= ~all;
      } while (clash != 0);
      same &= (1ull << lane) - 1ull;
      const int tile = __shfl(act, same != 0 ? 63 - __builtin_clzll(same) : lane);
      if (same != 0) old = tile;
    }
    const bool changed = may_write && act != old;
    const uint64_t changes = __builtin_amdgcn_ballot_w64(changed);
    auto first_steps = [](int k) { return k >= 64 ? ~0ull : (1ull << k) - 1ull; };
    const bool ends = t + 1 + lane >= a.max_steps ||
                      (a.max_changes > 0 && n_changes + (int)__popcll(changes & first_steps(lane + 1)) >= a.max_changes);
    const uint64_t end = a.autoreset ? __builtin_amdgcn_ballot_w64(lane < n && ends) : 0ull;
    const int used = end != 0 ? (int)__builtin_ctzll(end) + 1 : n;
    if (used != n) act_next = action_at(done_steps + used);
    // the edits, as far as the start of each span that lies among these steps
    for (int from = 0; from < used;) {
      const int to = span < sp.spans ? min(used, span * sp.steps - done_steps) : used;
      if (changed && lane >= from && lane < to) {
#pragma unroll
        for (int k = 0; k < PR::P; ++k)
          if (((old ^ act) >> k) & 1) atomicXor(&rows[k][word][y], 1u << (x & 31));
      }
      from = to;
      if (to == used) break;
      level_from_lds();
      store_span(span, (uint32_t)__builtin_amdgcn_readlane((int)after, to - 1), t + to, n_changes + (int)__popcll(changes & first_steps(to)));
      span += kSpanStartWaves;
    }
    t += used;
    n_changes += (int)__popcll(changes & first_steps(used));
    at = (uint32_t)__builtin_amdgcn_readlane((int)after, used - 1);
    done_steps += used;
    if (end != 0) {  // a new episode
      key = env_key(a.seed, (uint64_t)env, (uint64_t)(episode + 1));
      begin_episode<S, PROBLEM, true>(a, L, key, p, fz, h, w, py, px, true, env);
      h = __builtin_amdgcn_readfirstlane(h);
      w = __builtin_amdgcn_readfirstlane(w);
      at = (uint32_t)__builtin_amdgcn_readfirstlane((int)((uint32_t)py | (uint32_t)px << 8));
      episode += 1;
      t = 0;
      n_changes = 0;
      if ((a.ctrl_mask >> yi) & 1u) tg = control_target(a, key, yi);
      targets_moved = true;
      lds_sync();
      level_to_lds();
    }
    if (span < sp.spans && span * sp.steps == done_steps) {
      level_from_lds();
      store_span(span, at, t, n_changes);
      span += kSpanStartWaves;
    }
  }
  if (wave != 0) return;
  level_from_lds();
  if (primary) {
#pragma unroll
    for (int k = 0; k < PR::P; ++k) reinterpret_cast<W*>(a.planes)[(size_t)k * a.plane_stride + ridx] = p[k];
    reinterpret_cast<W*>(a.frozen)[ridx] = fz;
    if (targets_moved && L.y < PR::M) a.targets[(size_t)env * kMaxMetrics + L.y] = tg;
  }
  store_env(a.env + env, at, t, n_changes, L.gany((uint32_t)L.y == (at & 0xffu) && ((fz >> (at >> 8)) & 1) != 0) ? 1u : 0u);
}

// One span of the rollout for a group of levels: block x is the group, y the span.
template <int S, int PROBLEM>
__global__ __launch_bounds__(320) void rollout_span_kernel(KArgs a, SpanArgs sp) {
  using W = typename RowWord<S>::T;
  const int span = (int)blockIdx.y;
  const size_t level0 = (size_t)span * a.B, step0 = (size_t)span * sp.steps, out0 = step0 * a.B;
  a.planes = reinterpret_cast<W*>(sp.planes) + level0 * S;
  a.plane_stride = sp.plane_stride;
  a.frozen = reinterpret_cast<W*>(sp.frozen) + level0 * S;
  a.env = sp.env + level0;
  a.targets = sp.targets + level0 * kMaxMetrics;
  a.actions += out0;
  if (a.obs != nullptr) a.obs += out0 * (size_t)a.env_obs_bytes;
  if (a.reward != nullptr) a.reward += out0;
  if (a.done != nullptr) a.done += out0;
  a.rollout_steps = min(sp.steps, a.rollout_steps - (int)step0);
  step_body<S, PROBLEM, kModeSpan, true, kWidthAny>(a, span == sp.spans - 1);
}

// ------------------------------------------------- plain-layout conversion

// Levels in the plain layout (bytes [B][max_h][max_w]) -> bit-planes, and the metrics of what was
// installed, in one pass.  A wavefront takes the levels of its lane groups, whose cells are one
// contiguous run of bytes in either array: it reads the run in 16-byte pieces, packs each piece to 16 bits per plane with a multiply per four cells, and
// keeps the packed runs in LDS, out of which every lane then cuts its row.  Bound by latency and by
// the from-scratch metrics that follow.  Reading the bytes one by one, a thread per row, took
// 31 us for 5001 levels of 27x45 (12 MB) in a kernel of its own, and the metrics a second one
// (16 us); both together now take 18.
struct LevelSource {
  const int8_t* tiles;
  const uint8_t* frozen;  // or NULL: no pinpoints
  const int16_t *hw, *pos;
};
// bit 0 of every byte that is not zero
__device__ __forceinline__ uint32_t nonzero_bytes(uint32_t v) {
  return ((((v & 0x7f7f7f7fu) + 0x7f7f7f7fu) | v) >> 7) & 0x01010101u;
}
// bit 0 of the four bytes of v (whose other bits are zero), moved together
__device__ __forceinline__ uint32_t gather_nibble(uint32_t v) { return (v * 0x01020408u) >> 24; }
// The 16 bytes of an array from byte `at` on, for any address; what lies behind its `total` bytes
// is not read and reads as zero.
typedef u32x4 __attribute__((aligned(1))) unaligned_u32x4;
__device__ __forceinline__ u32x4 load_piece(const uint8_t* array, size_t at, size_t total) {
  if (at + 16 <= total) return *reinterpret_cast<const unaligned_u32x4*>(array + at);
  uint64_t lo = 0, hi = 0;
  if (total >= 16) {  // the last 16 bytes, moved down
    const u32x4 v = *reinterpret_cast<const unaligned_u32x4*>(array + total - 16);
    lo = (uint64_t)v.x | ((uint64_t)v.y << 32);
    hi = (uint64_t)v.z | ((uint64_t)v.w << 32);
    const int by = 8 * (int)(at + 16 - total);
    lo = by < 64 ? (lo >> by) | (hi << 1 << (63 - by)) : hi >> (by - 64);
    hi = by < 64 ? hi >> by : 0ull;
  } else {
#pragma unroll 1
    for (size_t j = total; j > at; --j) {
      hi = (hi << 8) | (lo >> 56);
      lo = (lo << 8) | array[j - 1];
    }
  }
  const u32x4 r = {(uint32_t)lo, (uint32_t)(lo >> 32), (uint32_t)hi, (uint32_t)(hi >> 32)};
  return r;
}

template <int S, int PROBLEM>
__device__ __forceinline__ void load_plain_rows(const KArgs& a, const Lanes<S>& L, const WaveMap<S>& wm, const LevelSource& src,
                                                int h, int w, typename RowWord<S>::T (&p)[Prob<PROBLEM>::P],
                                                typename RowWord<S>::T& fz) {
  using W = typename RowWord<S>::T;
  using PR = Prob<PROBLEM>;
  constexpr int kHalves = 64 * S / 16 + 4;  // (a row is cut out of three words)
  __shared__ __align__(4) uint16_t runs[PR::P + 1][kHalves];
  const int cells = a.max_h * a.max_w, n = wm.nvalid * cells;
  const size_t at0 = (size_t)wm.env0 * (size_t)cells, total = (size_t)a.B * (size_t)cells;
  const uint8_t* tiles = reinterpret_cast<const uint8_t*>(src.tiles);
  const bool with_fz = src.frozen != nullptr;
  u32x4 t = {0, 0, 0, 0}, f = {0, 0, 0, 0};
  auto request = [&](int q) {
    if (16 * q < n) {
      t = load_piece(tiles, at0 + 16 * q, total);
      if (with_fz) f = load_piece(src.frozen, at0 + 16 * q, total);
    }
  };
  request(L.lane);
#pragma unroll 1
  for (int q = L.lane; 16 * q < n; q += 64) {
    const uint32_t tw[4] = {t.x, t.y, t.z, t.w}, fw[4] = {f.x, f.y, f.z, f.w};
    request(q + 64);
    uint32_t bits[PR::P] = {}, fbits = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      // a code that is no tile of the problem counts as tile 0
      uint32_t bad = nonzero_bytes(tw[j] & (0x01010101u * (0xffu & ~((1u << PR::P) - 1u))));
      if constexpr (PR::K == 7) bad |= tw[j] & (tw[j] >> 1) & (tw[j] >> 2) & 0x01010101u;
#pragma unroll
      for (int i = 0; i < PR::P; ++i) bits[i] |= gather_nibble((tw[j] >> i) & 0x01010101u & ~bad) << (4 * j);
      fbits |= gather_nibble(nonzero_bytes(fw[j])) << (4 * j);
    }
#pragma unroll
    for (int i = 0; i < PR::P; ++i) runs[i][q] = (uint16_t)bits[i];
    runs[PR::P][q] = (uint16_t)fbits;
  }
  lds_sync();
  const int bit = wm.sl.slot * cells + L.y * a.max_w, word = bit >> 5, sh = bit & 31;  // where this lane's row starts
  const W mask = wm.valid ? inside_row<W>(L.y, h, w) : (W)0;
  auto row = [&](int i) -> W {
    const uint32_t* words = reinterpret_cast<const uint32_t*>(runs[i]) + word;
    uint64_t r = ((uint64_t)words[0] | ((uint64_t)words[1] << 32)) >> sh;
    if constexpr (S == 64) r |= (uint64_t)words[2] << 1 << (63 - sh);
    return (W)r & mask;
  };
  fz = 0;
#pragma unroll
  for (int i = 0; i < PR::P; ++i) p[i] = 0;
  if (mask != 0) {
#pragma unroll
    for (int i = 0; i < PR::P; ++i) p[i] = row(i);
    fz = row(PR::P);
  }
}

template <int S, int PROBLEM>
__global__ __launch_bounds__(64) void set_state_kernel(KArgs a, LevelSource src) {
  using W = typename RowWord<S>::T;
  using PR = Prob<PROBLEM>;
  Lanes<S> L;
  WaveMap<S> wm;
  wm.init(a, L, nullptr, (int)blockIdx.x, a.envs_per_wave_log2 & 0xff);
  const int16_t* hwp = src.hw + 2 * (size_t)wm.envl;
  const int16_t* qp = src.pos + 2 * (size_t)wm.envl;
  // the episode and its key stay (read as words: a struct that is loaded whole and then changed field
  // by field is kept in memory by the compiler, in LDS slots found through the dispatch packet, which
  // lies in host memory: 13 us of a launch)
  const uint4* erp = reinterpret_cast<const uint4*>(a.env + wm.envl);
  const uint4 er0 = erp[0], er1 = erp[1];
  const int h = min(max((int)hwp[0], 1), a.max_h), w = min(max((int)hwp[1], 1), a.max_w);
  const int py = min(max((int)qp[0], 0), h - 1), px = min(max((int)qp[1], 0), w - 1);
  W p[PR::P], fz;
  load_plain_rows<S, PROBLEM>(a, L, wm, src, h, w, p, fz);
  W* planes = reinterpret_cast<W*>(a.planes);
  const size_t ridx = (size_t)wm.envl * S + L.y;
  EnvRec er;
  er.episode = (int32_t)er0.w;
  er.key = (uint64_t)er1.x | ((uint64_t)er1.y << 32);
  er.pad_ = 0;
  er.h = (uint8_t)h;
  er.w = (uint8_t)w;
  er.py = (uint8_t)py;
  er.px = (uint8_t)px;
  er.t = 0;
  er.n_changes = 0;
  er.cell_frozen = L.gany(L.y == py && ((fz >> px) & 1)) ? 1u : 0u;
  if (wm.primary) {
#pragma unroll
    for (int i = 0; i < PR::P; ++i) planes[(size_t)i * a.plane_stride + ridx] = p[i];
    reinterpret_cast<W*>(a.frozen)[ridx] = fz;
    if (L.y == 0) a.env[wm.env] = er;
  }
  int m[PR::M];
  W comp;
  full_metrics<S, PROBLEM>(L, p, inside_row<W>(L.y, h, w), wm.valid, m, comp);
  if (wm.primary && L.y == 0) store_metrics<S, PROBLEM>(a.metrics + (size_t)wm.env * kMaxMetrics, m);
  if constexpr (PROBLEM == kBinary) {  // (the plane after the tile planes)
    if (wm.primary) planes[(size_t)PR::P * a.plane_stride + ridx] = comp;
  }
}

// Bit-planes -> the plain layout.  A thread writes 16 consecutive bytes of the tile array and of
// the pinpoint array, wherever rows and levels end in between: the bits of each row they touch
// (one or two rows for most widths) are put together and widened with a multiply per four cells.
// Bound by its stores and by how long a thread takes to reach them: everything that it reads of its first two
// rows, and of the level whose scalars it writes, is requested at once, and places are found without a
// division.  5001 levels of 27x45 (12 MB): a thread per row that wrote byte after byte took 49 us, one row
// after the other and divisions 7.5, this 5.8.
template <typename W, int P>
__global__ __launch_bounds__(kGetThreads) void get_state_kernel(KArgs a, int S, GetSizes sizes, int8_t* tiles, uint8_t* fro, int16_t* hw,
                                                                int16_t* pos, int32_t* counters) {
  const W* planes = reinterpret_cast<const W*>(a.planes);
  const GetPiece pc = get_piece(blockIdx.x, blockIdx.y, (int)threadIdx.x, sizes);
  const uint64_t e = get_level(blockIdx.x, blockIdx.y, (int)threadIdx.x);
  const bool scalars = e < (uint64_t)a.B && (hw || pos || counters);
  uint4 er = make_uint4(0, 0, 0, 0);
  if (scalars) er = *reinterpret_cast<const uint4*>(a.env + e);
  if (pc.n > 0 && (tiles || fro)) {
    const int n = pc.n;
    int env = pc.env, y = pc.y, x = pc.x;
    uint32_t bits[P] = {}, in = 0, fz = 0;
    struct Row {
      W p[P], fz;
      uint32_t hw;  // the first word of the level's record: height and width in the lower two bytes
    };
    auto request = [&](int env_, int y_) {
      Row r;
      const size_t row = (size_t)env_ * S + y_;
#pragma unroll
      for (int i = 0; i < P; ++i) r.p[i] = planes[(size_t)i * a.plane_stride + row];
      r.fz = reinterpret_cast<const W*>(a.frozen)[row];
      r.hw = *reinterpret_cast<const uint32_t*>(a.env + env_);
      return r;
    };
    auto add = [&](const Row& r, int y_, int x_, int run, int got) {
      const uint32_t mask = (1u << run) - 1u;
#pragma unroll
      for (int i = 0; i < P; ++i) bits[i] |= ((uint32_t)(r.p[i] >> x_) & mask) << got;
      fz |= ((uint32_t)(r.fz >> x_) & mask) << got;
      in |= ((uint32_t)(inside_row<W>(y_, (int)(r.hw & 0xffu), (int)((r.hw >> 8) & 0xffu)) >> x_) & mask) << got;
    };
    const int run0 = min(n, a.max_w - x), run1 = min(n - run0, a.max_w);
    const bool wraps = y + 1 == a.max_h;
    const int env1 = run1 > 0 && wraps ? env + 1 : env, y1 = run1 == 0 ? y : wraps ? 0 : y + 1;
    const Row r0 = request(env, y), r1 = request(env1, y1);
    add(r0, y, x, run0, 0);
    add(r1, y1, 0, run1, run0);
    env = env1;
    y = y1;
    for (int got = run0 + run1; got < n;) {  // (rows of less than 15 cells)
      if (++y == a.max_h) {
        y = 0;
        ++env;
      }
      const int run = min(n - got, a.max_w);
      add(request(env, y), y, 0, run, got);
      got += run;
    }
    // (a nibble times 0x204081 puts bit k at bit 8 k)
    auto widen = [](uint32_t b, int j) { return __umul24((b >> (4 * j)) & 15u, 0x00204081u) & 0x01010101u; };
    uint32_t t[4], f[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint32_t inj = widen(in, j), outj = inj ^ 0x01010101u;
      t[j] = (outj << 8) - outj;
#pragma unroll
      for (int i = 0; i < P; ++i) t[j] |= widen(bits[i] & in, j) << i;
      f[j] = widen(fz & in, j);
    }
    auto store = [&](uint8_t* dst, const uint32_t (&v)[4]) {
      dst += pc.at;
      if (n == kGetBytes && ((uintptr_t)dst & 15u) == 0) {
        *reinterpret_cast<uint4*>(dst) = make_uint4(v[0], v[1], v[2], v[3]);
      } else {
#pragma unroll
        for (int j = 0; j < kGetBytes; ++j)
          if (j < n) dst[j] = (uint8_t)(v[j >> 2] >> (8 * (j & 3)));
      }
    };
    if (tiles) store(reinterpret_cast<uint8_t*>(tiles), t);
    if (fro) store(fro, f);
  }
  if (scalars) {
    if (hw) {
      hw[2 * (size_t)e] = (int16_t)(er.x & 0xffu);
      hw[2 * (size_t)e + 1] = (int16_t)((er.x >> 8) & 0xffu);
    }
    if (pos) {
      pos[2 * (size_t)e] = (int16_t)((er.x >> 16) & 0xffu);
      pos[2 * (size_t)e + 1] = (int16_t)(er.x >> 24);
    }
    if (counters) {
      counters[3 * (size_t)e] = (int32_t)er.y;
      counters[3 * (size_t)e + 1] = (int32_t)er.z;
      counters[3 * (size_t)e + 2] = (int32_t)er.w;
    }
  }
}

__global__ void copy_metrics_kernel(const int32_t* src, int32_t* dst, int B, int M) {
  int idx = (int)(blockIdx.x * blockDim.x + threadIdx.x);
  if (idx >= B * M) return;
  dst[idx] = src[(size_t)(idx / M) * kMaxMetrics + idx % M];
}

__global__ void set_targets_kernel(const int32_t* src, uint32_t* dst, int B, int M) {
  int idx = (int)(blockIdx.x * blockDim.x + threadIdx.x);
  if (idx >= B * M) return;
  int env = idx / M, i = idx % M;
  dst[(size_t)env * kMaxMetrics + i] = pack_range(src[2 * idx], src[2 * idx + 1]);
}

__global__ void get_targets_kernel(const uint32_t* src, int32_t* dst, int B, int M) {
  int idx = (int)(blockIdx.x * blockDim.x + threadIdx.x);
  if (idx >= B * M) return;
  uint32_t t = src[(size_t)(idx / M) * kMaxMetrics + idx % M];
  dst[2 * idx] = (int32_t)(t & 0xffffu);
  dst[2 * idx + 1] = (int32_t)(t >> 16);
}

// The consumer's side of the bit-packed observation format: one workgroup per level turns the
// packed row back into one-hot elements of 1, 2 or 4 bytes (the value `one`, or zero).  The row is
// read once, 16 bytes a thread, into LDS, so that nothing but stores follows; the loads of three
// bytes a chunk, which short rows keep, hold the stores up.  The output of a level is written as
// aligned 16-byte chunks, with the few elements before the first and after the last full chunk one
// by one; each chunk needs the 16, 8 or 4 bits that start at its first cell.  Bound by the stores:
// 8192 levels of 4805 cells to 1 / 2 / 4 bytes 10.2 / 15.2 / 35.7 -> 8.0 / 13.4 / 31.9 us.
template <int ES, bool STAGED>  // element size in bytes; row through LDS
__global__ __launch_bounds__(256) void unpack_obs_kernel(const uint8_t* packed, int64_t packed_stride, uint8_t* out,
                                                        int32_t cells, uint32_t one) {
  constexpr int PER = 16 / ES;  // elements per 16-byte chunk
  __shared__ u32x4 bits16[(kMaxPackedRow + 15) / 16 + 1];  // the row, and room for the word after the last one
  const uint32_t* const bits = reinterpret_cast<const uint32_t*>(bits16);
  const int t = (int)threadIdx.x, T = (int)blockDim.x;
  const int64_t level = blockIdx.x;
  const uint8_t* row = packed + level * packed_stride;
  uint8_t* dst = out + level * (int64_t)cells * ES;
  const int row_bytes = (cells + 7) >> 3;
  if constexpr (STAGED) {
    for (int i = t; i * 16 < row_bytes; i += T) bits16[i] = load_piece(row, (size_t)i * 16, (size_t)row_bytes);
    __syncthreads();
  }
  // PER bits and more that start at cell e, which is bit e % 32 of word e / 32
  auto bits_at = [&](int e) -> uint32_t {
    if constexpr (STAGED) return __builtin_amdgcn_alignbit(bits[(e >> 5) + 1], bits[e >> 5], (uint32_t)e & 31u);
    const int b0 = e >> 3;  // (reads stay inside the row)
    uint32_t v = row[b0];
    if (b0 + 1 < row_bytes) v |= (uint32_t)row[b0 + 1] << 8;
    if (b0 + 2 < row_bytes) v |= (uint32_t)row[b0 + 2] << 16;
    return v >> (e & 7);
  };
  auto store_one = [&](int e) {
    const uint32_t bit = STAGED ? (bits[e >> 5] >> (e & 31)) & 1u : (row[e >> 3] >> (e & 7)) & 1u;
    if constexpr (ES == 1) dst[e] = (uint8_t)(bit ? one : 0u);
    else if constexpr (ES == 2) reinterpret_cast<uint16_t*>(dst)[e] = (uint16_t)(bit ? one : 0u);
    else reinterpret_cast<uint32_t*>(dst)[e] = bit ? one : 0u;
  };
  const int head = min(cells, (int)(((16u - (uint32_t)((uintptr_t)dst & 15u)) & 15u) / ES));  // elements before the first aligned chunk
  const int nchunks = (cells - head) / PER;
  const int tail0 = head + nchunks * PER;
  if (t < head) store_one(t);
  if (tail0 + t < cells) store_one(tail0 + t);
  for (int c = t; c < nchunks; c += T) {
    const int e = head + c * PER;
    const uint32_t b = bits_at(e);
    u32x4 v;
    if constexpr (ES == 1) {
      // a nibble times 0x204081 puts bit k at bit 8 k (0, 7, 14, 21 are shifted copies)
      v.x = (__umul24(b & 15u, 0x00204081u) & 0x01010101u) * one;
      v.y = (__umul24((b >> 4) & 15u, 0x00204081u) & 0x01010101u) * one;
      v.z = (__umul24((b >> 8) & 15u, 0x00204081u) & 0x01010101u) * one;
      v.w = (__umul24((b >> 12) & 15u, 0x00204081u) & 0x01010101u) * one;
    } else if constexpr (ES == 2) {
      auto two = [&](uint32_t q) { return ((q & 1u) ? one : 0u) | ((q & 2u) ? one << 16 : 0u); };
      v.x = two(b);
      v.y = two(b >> 2);
      v.z = two(b >> 4);
      v.w = two(b >> 6);
    } else {
      v.x = (b & 1u) ? one : 0u;
      v.y = (b & 2u) ? one : 0u;
      v.z = (b & 4u) ? one : 0u;
      v.w = (b & 8u) ? one : 0u;
    }
    *reinterpret_cast<u32x4*>(dst + (int64_t)e * ES) = v;
  }
}

// Measurement aid: nothing but stores, in the pattern of the observation writer (one wavefront per
// contiguous region, aligned 16-byte stores, 1 KiB per wavefront instruction; with by_die the
// regions are dealt to the workgroups the way a rollout deals its level groups, see
// level_group_of_block) or, with `linear`, as one sweep over the whole buffer (wavefront w writes
// the 1 KiB pieces w, w + n, w + 2n, ...).  What it sustains is the store rate that the step
// kernels can be held against.
__global__ __launch_bounds__(64) void store_rate_kernel(uint8_t* dst, int64_t n_regions, int32_t region_bytes,
                                                        int32_t mode, int32_t linear, int32_t by_die) {
  const int lane = (int)(threadIdx.x & 63u);
  const int64_t w = level_group_of_block<true>(by_die), n = gridDim.x;
  const int chunks = region_bytes >> 4;  // 16-byte chunks per region
  const u32x4 v = {0x01010101u, 0x00010001u, 0x01000100u, (uint32_t)w};
  for (int64_t r = w; r < n_regions; r += n) {
    for (int q = lane; q < chunks; q += 64) {
      const int64_t piece = q >> 6;  // which 1 KiB piece of the region
      const int64_t off = linear ? ((piece * n_regions + r) << 10) + ((int64_t)(q & 63) << 4)
                                 : r * (int64_t)region_bytes + ((int64_t)q << 4);
      u32x4* at = reinterpret_cast<u32x4*>(dst + off);
      if (mode == kStoreThrough) {
        asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 0" ::"v"(at), "v"(v) : "memory");
      } else if (mode == kStoreStream) {
        __builtin_nontemporal_store(v, at);
      } else {
        *at = v;
      }
    }
  }
}

// Cross-lane exchange check: the DPP shifts against the plain shuffle definition.
__global__ __launch_bounds__(64) void selftest_kernel(int32_t* mismatches) {
  int lane = (int)(threadIdx.x & 63u);
  uint32_t v32 = 0x9E3779B9u * (uint32_t)(lane + 1);
  uint64_t v64 = mix64((uint64_t)lane + 17);
  int bad = 0;
  {
    Lanes<16> L;
    uint32_t up = __shfl_up(v32, 1), dn = __shfl_down(v32, 1);
    bad += L.from_above(v32) != (L.y == 0 ? 0u : up);
    bad += L.from_below(v32) != (L.y == 15 ? 0u : dn);
  }
  {
    Lanes<32> L;
    uint32_t up = __shfl_up(v32, 1), dn = __shfl_down(v32, 1);
    bad += L.from_above(v32) != (L.y == 0 ? 0u : up);
    bad += L.from_below(v32) != (L.y == 31 ? 0u : dn);
  }
  {
    Lanes<64> L;
    uint64_t up = __shfl_up(v64, 1), dn = __shfl_down(v64, 1);
    bad += L.from_above(v64) != (L.y == 0 ? 0ull : up);
    bad += L.from_below(v64) != (L.y == 63 ? 0ull : dn);
  }
  // group reductions against a plain shuffle butterfly
  int iv = (int)(v32 >> 20) - 1000;
  {
    Lanes<16> L;
    int sum = iv, mx = iv;
    for (int o = 8; o > 0; o >>= 1) { sum += __shfl_xor(sum, o); mx = max(mx, __shfl_xor(mx, o)); }
    bad += L.gsum(iv) != sum;
    bad += L.gmax(iv) != mx;
  }
  {
    Lanes<32> L;
    int sum = iv, mx = iv;
    for (int o = 16; o > 0; o >>= 1) { sum += __shfl_xor(sum, o); mx = max(mx, __shfl_xor(mx, o)); }
    bad += L.gsum(iv) != sum;
    bad += L.gmax(iv) != mx;
  }
  {
    Lanes<64> L;
    int sum = iv, mx = iv;
    for (int o = 32; o > 0; o >>= 1) { sum += __shfl_xor(sum, o); mx = max(mx, __shfl_xor(mx, o)); }
    bad += L.gsum(iv) != sum;
    bad += L.gmax(iv) != mx;
  }
  if (bad) atomicAdd(mismatches, bad);
}

}  // namespace pcgrl

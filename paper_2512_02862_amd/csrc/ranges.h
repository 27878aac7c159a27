// Moves of rows by up to 256 destinations in two kernels over the same ranges:
// the rows' tiles are split into at most 512 contiguous ranges, one a block; a
// counting kernel leaves each range's count per destination, and the moving
// kernel adds up what lies before its range and then walks its tiles.
#pragma once

#include "pyst_internal.h"

namespace pyst {

constexpr int kRangeDigits = 256;
constexpr int kRangeParts = 512;
constexpr int kRangeGroup = 16, kRangeGroups = kRangeParts / kRangeGroup;
constexpr int kRangeThreads = 1024;

// Counts per destination: of each range, and of each group of 16 ranges (a row
// set per pass, cleared before the counting kernels).
struct RangeCounts {
  uint32_t *part;
  uint32_t *group;
  int ngroups;
  __device__ __forceinline__ uint32_t *of_part(int64_t p) const { return part + p * kRangeDigits; }
  __device__ __forceinline__ uint32_t *of_group(int pass, int64_t g) const {
    return group + (int64_t{pass} * ngroups + g) * kRangeDigits;
  }
};

inline int range_parts(int64_t n, int64_t tile) {
  return static_cast<int>(std::min<int64_t>(kRangeParts, std::max<int64_t>(1, ceil_div(n, tile))));
}

// Words of the counts of `parts` ranges (host), and their layout at `mem`.
inline size_t range_count_words(int parts, int passes) {
  return (static_cast<size_t>(parts) + static_cast<size_t>(passes) * ceil_div(parts, kRangeGroup)) * kRangeDigits;
}
inline RangeCounts range_counts_at(void *mem, int parts) {
  RangeCounts c;
  c.part = static_cast<uint32_t *>(mem);
  c.group = c.part + int64_t{parts} * kRangeDigits;
  c.ngroups = static_cast<int>(ceil_div(parts, kRangeGroup));
  return c;
}

// The tiles [t0, t1) of this block's range of n rows; neighbouring ranges run on
// one XCD.  False for blocks past the last range.
__device__ __forceinline__ bool range_of_block(int64_t n, int64_t tile, int64_t &part, int64_t &t0, int64_t &t1) {
  const int64_t tiles = (n + tile - 1) / tile, parts = tiles < kRangeParts ? tiles : kRangeParts;
  if (blockIdx.x >= parts) return false;
  part = xcd_block(blockIdx.x, parts);
  t0 = tiles * part / parts;
  t1 = tiles * (part + 1) / parts;
  return true;
}

struct RangeOffsets {
  static constexpr int G = kRangeThreads / kRangeDigits;
  uint32_t all[G][kRangeDigits], before[G][kRangeDigits];
};

// s_next[d]: where the first row of destination d in range `part` goes.  Called
// by 1024 threads; the caller synchronizes before reading s_next.  Returns (in
// wave 0) the number of rows moved in all.
__device__ __forceinline__ int64_t range_offsets(const RangeCounts &counts, int pass, int part, RangeOffsets &s,
                                                 int64_t *s_next) {
  constexpr int G = RangeOffsets::G;
  const int tid = static_cast<int>(threadIdx.x), lane = lane_id();
  const int d = tid % kRangeDigits, g = tid / kRangeDigits, group = part / kRangeGroup;
  uint32_t all = 0, before = 0;  // four threads a destination
#pragma unroll
  for (int j = 0; j < kRangeGroups / G; ++j) {
    const uint32_t c = j * G + g < counts.ngroups ? counts.of_group(pass, j * G + g)[d] : 0;
    all += c;
    before += j * G + g < group ? c : 0;
  }
#pragma unroll
  for (int j = 0; j < kRangeGroup / G; ++j) {
    const int p = group * kRangeGroup + j * G + g;
    before += p < part ? counts.of_part(p)[d] : 0;
  }
  s.all[g][d] = all;
  s.before[g][d] = before;
  __syncthreads();
  int64_t total = 0;
  if (tid < kWave) {  // exclusive scan over the destinations, four a lane
    int64_t a[4], la = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      a[j] = 0;
#pragma unroll
      for (int q = 0; q < G; ++q) a[j] += s.all[q][lane * 4 + j];
      la += a[j];
    }
    const int64_t incl = wave_inclusive_scan(la);
    int64_t ra = incl - la;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      int64_t at = ra;
#pragma unroll
      for (int q = 0; q < G; ++q) at += s.before[q][lane * 4 + j];
      s_next[lane * 4 + j] = at;
      ra += a[j];
    }
    total = __shfl(incl, kWave - 1);
  }
  return total;
}

}  // namespace pyst

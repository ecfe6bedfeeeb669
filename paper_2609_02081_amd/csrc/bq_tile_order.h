// Order of output tiles over the blocks of a launch (the split forms and the
// one-launch products).
#pragma once

#include "bq_internal.h"

namespace bq {

// Blocks are dealt to the 8 XCDs in turn (b % 8).  Position of block b among
// the blocks [p0, p1) of a launch when each XCD takes a contiguous run of
// positions.
__host__ __device__ __forceinline__ int64_t xcd_position(int64_t b, int64_t p0, int64_t p1) {
  const int64_t x = b & 7;
  // Blocks below p whose XCD precedes x; blocks of XCD x below p0.
  auto before = [&](int64_t p) { return (p >> 3) * x + ((p & 7) < x ? (p & 7) : x); };
  return before(p1) - before(p0) + (b >> 3) - ((p0 + 7 - x) >> 3);
}

// Tile t of an output, in groups of 8 tile rows (as in the FP64 GEMM).
__host__ __device__ __forceinline__ void grouped_tile(int t, int tiles_m, int tiles_n, int& tm, int& tn) {
  const int per_group = 8 * tiles_n, group = t / per_group, first_m = group * 8;
  const int gm = tiles_m - first_m < 8 ? tiles_m - first_m : 8, in_g = t - group * per_group;
  tm = first_m + in_g % gm;
  tn = in_g / gm;
}

}  // namespace bq

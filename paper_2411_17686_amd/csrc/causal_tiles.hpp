// Orders of the workgroups of causal maps.  (Host code too: what a test may ask.)
#pragma once
#include "common.hpp"

namespace ficoco {

// Row normalisers: one group of queries of every head after the other, those that see most keys first, instead of head by head.  Only where the first
// group sees at most three fifths of the keys that the last one does: else there is little to even out, and what the groups of a head share is
// read again for each (16 x (64 + 200) queries, 40 heads of 128: both kernels 58.3 us head by head, 64.1 so).  Over 700 shapes, head by head relative to
// this: up to 0.3 of the keys 1.09, 0.3 to 0.5 1.06, 0.5 to 0.6 1.025, 0.6 to 0.7 1.01 (at worst 0.94), beyond 1.00 (0.91).
inline bool causal_long_first(int keys_of_first, int keys_of_last) { return 5 * (int64_t)keys_of_first <= 3 * (int64_t)keys_of_last; }

// Head mean: the tiles that hold a key some query sees first, last queries first, then the others, which are zero.  Whole tiles, above kCausalTiles (where every tile has a place at once there is nothing to gain) and up to kCausalKeyTiles key tiles; with
// more, the keys of a group are more rows than the L2 of an XCD holds for the workgroups that share them.  Stage in columns relative to live first
// by key tiles, over 3000 calls: 5 to 11 1.02 to 1.04 (at worst 0.91), 12 and 13 1.02 (0.82: 6 x (768 + 200) queries), 14 to 17 1.00, 18 0.99 (0.81).
constexpr int kCausalTiles = 256, kCausalKeyTiles = 11;
__host__ __device__ __forceinline__ bool causal_live_first(int units, int k_tiles) { return units > kCausalTiles && k_tiles <= kCausalKeyTiles; }

// The largest m with m (m + 1) / 2 <= x.
__host__ __device__ __forceinline__ int triangle_row(int x) {
  int m = (int)((__builtin_sqrtf(8.0f * (float)x + 1.0f) - 1.0f) * 0.5f);
#ifdef __HIP_DEVICE_COMPILE__
  m = __builtin_amdgcn_readfirstlane(m);      // uniform
#endif
  if ((m + 1) * (m + 2) / 2 <= x) ++m;        // (a root rounded up or down)
  if (m * (m + 1) / 2 > x) --m;
  return m;
}

// Tile number `unit` of an image of groups x k_tiles in that order: group g of queries, key tile kt.  The first `full` groups hold only queries of the
// causal span, `per` key tiles long each: group g sees its first per (g + 1) key tiles.  The others see all.  In closed form: with a search over the groups
// in every workgroup 16 x (1152 + 300) queries of one head took 49.8 us (two kernels), 45.3 in the order of other maps.
__host__ __device__ __forceinline__ void causal_tile(int unit, int groups, int k_tiles, int per, int full, int& g, int& kt) {
  const int rest = (groups - full) * k_tiles, seen = rest + per * (full * (full + 1) / 2);
  if (unit < rest) {
    g = groups - 1 - unit / k_tiles;
    kt = unit % k_tiles;
  } else if (unit < seen) {                   // rows of a triangle, from its last one up
    const int left = seen - 1 - unit;
    g = triangle_row(left / per);
    kt = per * ((g + 1) * (g + 2) / 2) - 1 - left;
  } else {                                    // key tiles that no such group sees, then the triangle's other half
    const int dead = unit - seen, wide = k_tiles - per * full, left = dead - full * wide;
    if (left < 0) {
      g = dead / wide;
      kt = per * full + dead % wide;
    } else {
      const int t = triangle_row(left / per);
      g = full - 2 - t;
      kt = per * (g + 1) + left - per * (t * (t + 1) / 2);
    }
  }
}

}  // namespace ficoco

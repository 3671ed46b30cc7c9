// The lists of (item, tile) pairs that the workgroups of seq_grad_walk.hip walk: integer arithmetic only, also for the host.
#pragma once

#include <hip/hip_runtime.h>

namespace isopo {

// Division of a tile index by a number the host knows: floor(n / d) is floor(n * mul / 2^32) or one more, mul = floor(2^32 / d).
struct TileDiv {
  unsigned d, mul;
};
inline TileDiv tile_div_by(unsigned d) { return {d, d > 1 ? (unsigned)((1ull << 32) / d) : 0xffffffffu}; }
__host__ __device__ __forceinline__ int tile_div(int n, TileDiv v) {
  unsigned q = (unsigned)(((unsigned long long)(unsigned)n * v.mul) >> 32);
  if ((unsigned)n - q * v.d >= v.d) ++q;
  return (int)q;
}

// A workgroup's way through the list of (item, tile) pairs, items being sequences (or the one sum over all tokens), in one of
// three arrangements (plan_walk says which, and why):
//   dealt   every item's tiles go to the XCDs in contiguous eighths, the odd tiles of a count that is no multiple of eight to one
//           XCD after the other, on from item to item
//   ranges  XCD x takes the pairs first .. end of the item-major list
//   single  the same ranges, with a workgroup for every pair
// Workgroup w of an XCD's W takes pairs w, 2W-1-w, 2W+w, 4W-1-w ... of the XCD's list: with the sequences sorted by length
// nobody is left with a long one at the end.  Of pairs that outlast what the others have to do, `alone`, each has a workgroup to
// itself, and the others walk the rest of the list.
enum WalkKind { kDealt, kRanges, kSingle };

template <int KIND>
struct PairWalk {
  int x, w, W, tiles, items;
  TileDiv by_tiles;
  int end;
  int i, e, turn;                        // item; place in the XCD's share of the item (dealt) or in the list
  __host__ __device__ __forceinline__ int share(int item) const {
    return (tiles >> 3) + (((x - item * (tiles & 7)) & 7) < (tiles & 7) ? 1 : 0);
  }
  __host__ __device__ __forceinline__ void settle() {
    if constexpr (KIND != kDealt) {
      i = e < end ? tile_div(e, by_tiles) : items;
    } else {
      while (i < items && e >= tiles) { e -= tiles; i += 8; }    // an XCD's share of eight items is `tiles`
      while (i < items && e >= share(i)) { e -= share(i); ++i; }
    }
#ifdef __HIP_DEVICE_COMPILE__
    if constexpr (KIND != kDealt) i = __builtin_amdgcn_readfirstlane(i);       // a scalar register
#endif
  }
  __host__ __device__ __forceinline__ PairWalk(int workgroup, int per_xcd, int tiles_, int items_, TileDiv by_tiles_, int first,
                                               int end_, int alone) {
    tiles = tiles_; items = items_; by_tiles = by_tiles_; end = end_;
    x = workgroup & 7; w = workgroup >> 3; W = per_xcd;
    i = 0; e = first + w; turn = 0;
    if (KIND != kSingle && alone > 0) {
      W = w < alone ? 1 << 28 : W - alone;                       // the next pair: past the end of any list
      w = w < alone ? 0 : w - alone;
    }
    settle();
  }
  __host__ __device__ __forceinline__ void next() {
    if constexpr (KIND == kSingle) {
      i = items;
    } else {
      e += turn ? 2 * w + 1 : 2 * (W - w) - 1;
      turn ^= 1;
      settle();
    }
  }
  __host__ __device__ __forceinline__ bool more() const { return i < items; }
  __host__ __device__ __forceinline__ int tile() const {
    if constexpr (KIND != kDealt) return e - i * tiles;
    const int rest = tiles & 7, y = (x - i * rest) & 7;
    return y * (tiles >> 3) + (y < rest ? y : rest) + e;
  }
};

}  // namespace isopo

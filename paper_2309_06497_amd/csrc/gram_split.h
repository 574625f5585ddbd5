// How the Gram matrix of an unfolding d x K of a tensor block is cut into ranges of k (host only).
//
// It is a tile or a few per block over a long k, which leaves most of the CUs idle.  k is cut into
// ranges of at least 64, multiples of the slab depth, until there are about four workgroups per CU;
// their Gram matrices go, in float64, through scratch that holds `room` matrices of d x d per block, and are
// added there.  The blocks of ResNet-50, most of them 128 x 1152 twice: 706 us whole, 290 us cut.
#pragma once
#include <algorithm>
#include <cstdint>

namespace shampoo {

struct GramSplit { int32_t ranges, range; };   // ranges * range >= K, (ranges - 1) * range < K

// workgroups: of the launch without a split (tiles of all blocks); slab: what a range is a multiple of.
inline GramSplit gram_split(int64_t K, int64_t room, int64_t workgroups, int32_t slab) {
  const int64_t want = (1024 + workgroups - 1) / workgroups;
  const int64_t most = std::min({want, room, K / 64});
  if (most <= 1) return {1, (int32_t)K};
  // at least K / most values to a range, so that rounding the range up can only lower the number of ranges
  const int64_t range = ((K + most - 1) / most + slab - 1) / slab * slab;
  return {(int32_t)((K + range - 1) / range), (int32_t)range};
}

}  // namespace shampoo

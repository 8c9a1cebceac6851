// Grids of the persistent launches and the work items of a branching call (host
// arithmetic only).
#pragma once
#include <stdint.h>

#include <algorithm>
#include <vector>

#include "pdd_internal.hpp"
#include "pdd_tuning.hpp"

namespace pdd {

// Blocks of a persistent launch: as many per compute unit as asked for, but no
// more than it holds at a time (`held`, where wavefronts start on items of
// their own; else 0) and no more than there are items for.
inline int persistent_grid(int blocks_per_cu, int held, int n_items, int n_cus) {
  const int per_cu = held > 0 ? std::min(held, blocks_per_cu) : blocks_per_cu;
  const int per = kBlock / kWave, need = n_items / per + (n_items % per != 0 ? 1 : 0);
  return std::max(1, std::min(per_cu * n_cus, need));
}

// A branching call's items: about a point's last eighth in items of `small`
// trees, the rest in items of `big`.
inline TreeItems tree_items(int64_t n_points, int64_t trees, int64_t big, int64_t small) {
  TreeItems t{};
  t.n_points = (int32_t)n_points;
  t.trees = (uint32_t)trees;
  for (;; big *= 2, small *= 2) {
    big = std::min<int64_t>(big, 1ll << 31);   // (sizes are 32 bits; a point has fewer trees)
    small = std::min(small, big);
    const int64_t n_big = trees > big && small < big ? (trees - trees / 8) / big : 0;
    const int64_t n_small = (trees - n_big * big + small - 1) / small;
    if (n_points * (n_big + n_small) > (int64_t)INT32_MAX) continue;   // (slots are 32 bits)
    t.n_big = (int32_t)n_big;
    t.n_small = (int32_t)n_small;
    t.big = (uint32_t)big;
    t.small = (uint32_t)small;
    return t;
  }
}

inline std::vector<int64_t> first_slots(const TreeItems& t) {
  std::vector<int64_t> first((size_t)t.n_points + 1);
  for (size_t i = 0; i < first.size(); ++i) first[i] = (int64_t)i * (t.n_big + t.n_small);
  return first;
}

// The items of a branching call with a boundary.  An item size in the call's
// options is taken as it is.  Else trees stream across a wavefront's items, so
// short items cost it little and even out the wavefronts' ends: an eighth of a
// wavefront's share, from one tree per lane to 256 or the schedule table's size
// (1024 points x 10000 trees, 11 times: 33.0 ms with items of 2048, 28.7 of
// 512, 26.6 of 256; 27.0 with 64, whose sums and queue pops show).  Every item
// keeps a partial of 48 bytes per output time, so a large call's items grow
// with it: kBvpItemsPerWave of them even out the wavefronts' ends as well as
// more would (1024 points x 100000 trees: 229.9 ms and 70 MB of partials with
// items of 1024, 229.8 ms and 290 MB with 256).
constexpr int64_t kBvpItem = 256, kBvpItemsPerWave = 32;

inline TreeItems bvp_items(int64_t n_points, int64_t trees, const Tuning& t, int n_cus) {
  if (t.chunk_from == kChunkOption)
    return tree_items(n_points, trees, t.chunk_paths, std::max(std::min(256, t.chunk_paths), t.chunk_paths / 8));
  const int64_t total = n_points * trees, waves = (int64_t)n_cus * 16;
  int64_t big = t.chunk_from == kChunkTable ? t.chunk_paths : kBvpItem;
  big = std::min(big, std::max<int64_t>(kWave, total / (8 * waves)));
  while (total / big > kBvpItemsPerWave * waves) big *= 2;
  return tree_items(n_points, trees, big, std::max<int64_t>(kWave, big / 8));
}

}  // namespace pdd

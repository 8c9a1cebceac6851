// Host-only check of the work items that a call is cut into.  Reads one
// command a line from standard input and prints one line for each:
//   trees <points> <trees> <big> <small>        tree_items
//   bvp <points> <trees> <chunk> <from> <cus>   bvp_items (from: 0 default, 1 table, 2 option)
//   grid <blocks a CU> <held> <items> <cus>     persistent_grid
//   groups <n>                                  threads of a launch with a wavefront per group
// The answer of the first two is "<items a point> <big> <small> <covered>":
// covered is 1 if TreeItems::at deals every tree of every point out exactly
// once and every slot once (0 if it does not, -1 if there are too many items
// to look); that of the others is one number.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <iostream>
#include <sstream>
#include <string>
#include <vector>

#include "pdd_kernels.hpp"
#include "work_items.hpp"

using namespace pdd;

static int covered(const TreeItems& t) {
  if (t.count() > 5000000) return -1;
  const std::vector<int64_t> first = first_slots(t);
  std::vector<char> slot((size_t)t.count(), 0);
  std::vector<int64_t> trees((size_t)t.n_points, 0);
  std::vector<std::vector<char>> seen((size_t)t.n_points);
  for (int i = 0; i < t.count(); ++i) {
    const WorkItem w = t.at((uint32_t)i);
    if (w.node < 0 || w.node >= t.n_points || w.count == 0) return 0;
    if (w.slot < first[(size_t)w.node] || w.slot >= first[(size_t)w.node + 1] || slot[(size_t)w.slot]++) return 0;
    if ((uint64_t)w.p0 + w.count > t.trees) return 0;
    trees[(size_t)w.node] += w.count;
    if (t.trees <= 100000 && t.n_points <= 16) {
      std::vector<char>& s = seen[(size_t)w.node];
      s.resize(t.trees, 0);
      for (uint32_t k = 0; k < w.count; ++k)
        if (s[w.p0 + k]++) return 0;
    }
  }
  for (int64_t n : trees)
    if (n != (int64_t)t.trees) return 0;
  return 1;
}

int main() {
  std::string line;
  while (std::getline(std::cin, line)) {
    std::istringstream in(line);
    std::string what;
    int64_t points, trees, a, b, cus = 0;
    in >> what >> points;
    if (what == "groups") {
      std::cout << (int64_t)group_blocks(points) * kBlock << std::endl;
      continue;
    }
    if (what == "grid") {
      in >> trees >> a >> b;
      std::cout << persistent_grid((int)points, (int)trees, (int)a, (int)b) << std::endl;
      continue;
    }
    in >> trees >> a >> b;
    TreeItems t{};
    if (what == "trees") {
      t = tree_items(points, trees, a, b);
    } else {
      in >> cus;
      Tuning u{};
      u.chunk_paths = (int)a;
      u.chunk_from = (ChunkFrom)b;
      t = bvp_items(points, trees, u, (int)cus);
    }
    std::cout << (int64_t)t.n_big + t.n_small << ' ' << t.big << ' ' << t.small << ' ' << covered(t) << std::endl;
  }
  return 0;
}

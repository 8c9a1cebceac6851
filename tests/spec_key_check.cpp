// Host-only: the keys of the problem-specialised kernels' caches.  Prints, for
// a branching and for a walk kernel, the sizes of the two keys and of the
// generated source, and which embedded headers the key on disk holds.
#include <cstdio>
#include <string>

#include "pdd_spec.hpp"

namespace pdd {
extern const int kRtcHeaderCount;
extern const char* const kRtcHeaderNames[];
extern const char* const kRtcHeaderBodies[];
}

using namespace pdd;

int main() {
  for (int walk = 0; walk < 2; ++walk) {
    const std::string src = walk ? spec_walk_source("struct T {};") : spec_branch_source("struct T {};");
    const std::string name = walk ? spec_walk_name(true, 2, 3, RNG_QUAD24, false)
                                  : spec_branch_name(true, 1, RNG_QUAD24, true);
    const std::string file = spec_file_key("gfx950", name, src);
    std::printf("%s %zu %zu", walk ? "walk" : "branch", name.size() + src.size(), spec_table_key(0, name, src).size());
    for (int i = 0; i < kRtcHeaderCount; ++i)
      if (file.find(kRtcHeaderBodies[i]) != std::string::npos) std::printf(" %s", kRtcHeaderNames[i]);
    std::printf("\n");
    if (spec_table_key(0, name, src) == spec_table_key(1, name, src) ||
        spec_table_key(0, name, src) == spec_table_key(0, name, src + " ") ||
        spec_table_key(0, name, src) == spec_table_key(0, name + " ", src) ||
        file == spec_file_key("gfx942", name, src) || file == spec_file_key("gfx950", name, src + " "))
      return 1;
  }
  return 0;
}

// Prints what the launch rules choose for the argument list: router T N d (slices steps token-blocks groups row-blocks),
// few d I elem T (1 if up to 15 tokens stream their experts), batch d I elem rows used items
// tiles (1 if a token batch does).
#include <cstdio>
#include <cstdlib>
#include <cstring>

#include "router_rules.hpp"
#include "stream_rules.hpp"

int main(int argc, char** argv) {
  for (int i = 1; i < argc;) {
    if (!std::strcmp(argv[i], "router") && i + 3 < argc) {
      const wisp::RouterTiles r = wisp::router_tiles(std::atoi(argv[i + 1]), std::atoi(argv[i + 2]), std::atoi(argv[i + 3]));
      std::printf("%d %d %d %d %d\n", r.slices, r.steps, r.tb, r.groups, r.rb);
      i += 4;
    } else if (!std::strcmp(argv[i], "few") && i + 4 < argc) {
      std::printf("%d\n", wisp::stream_few_tokens(std::atoi(argv[i + 1]), std::atoi(argv[i + 2]), std::atoi(argv[i + 3]), std::atoi(argv[i + 4])));
      i += 5;
    } else if (!std::strcmp(argv[i], "batch") && i + 7 < argc) {
      std::printf("%d\n", wisp::stream_batch(std::atoi(argv[i + 1]), std::atoi(argv[i + 2]), std::atoi(argv[i + 3]), std::atoi(argv[i + 4]),
                                             std::atoi(argv[i + 5]), std::atoi(argv[i + 6]), std::atoi(argv[i + 7])));
      i += 8;
    } else {
      return 2;
    }
  }
  return 0;
}

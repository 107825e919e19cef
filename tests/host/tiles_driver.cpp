// Prints the similarity kernel's tile side and work list for prompts of the given sizes: one
// "first-row first-column end" line per entry.
#include "equiv_tiles.hpp"

#include <cstdio>
#include <cstdlib>

int main(int argc, char** argv) {
  std::vector<int2> prompts;
  int at = 0;
  for (int i = 1; i < argc; ++i) {
    const int n = std::atoi(argv[i]);
    prompts.push_back(make_int2(at, at + n));
    at += n;
  }
  const ga::EquivTiles tiles = ga::equiv_tiles(prompts);
  std::printf("%d\n", tiles.tile);
  for (const int4& t : tiles.items) std::printf("%d %d %d\n", t.x, t.y, t.z);
  return 0;
}

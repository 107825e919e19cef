// Prints the similarity kernel's work list for prompts of the given sizes: one "first-row
// first-column end" line per entry.
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
  for (const int4& t : ga::equiv_tiles(prompts)) std::printf("%d %d %d\n", t.x, t.y, t.z);
  return 0;
}

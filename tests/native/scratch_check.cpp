// alloc_most against allocators with a given amount of room: prints, for every
// (want, least, room), the amount obtained.
#include <cstdio>

#include "host/scratch.h"

int main() {
  const size_t cases[][3] = {{512, 1, 512}, {512, 1, 511}, {512, 1, 100}, {512, 1, 1}, {512, 1, 0}, {512, 64, 40},
                             {1, 1, 1}, {1, 1, 0}, {0, 1, 9}, {7, 1, 3}};
  for (const auto& c : cases) {
    size_t asked = 0, calls = 0;
    const size_t got = tmcs::alloc_most(c[0], c[1], [&](size_t n) { ++calls; asked = n; return n <= c[2]; });
    if (got && asked != got) return 1;
    std::printf("%zu %zu %zu %zu %zu\n", c[0], c[1], c[2], got, calls);
  }
  return 0;
}

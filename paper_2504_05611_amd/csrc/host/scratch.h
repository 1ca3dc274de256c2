// Sizes of scratch that a call can do with less of.
#pragma once

#include <cstddef>

namespace tmcs {

// The largest of want, want / 2, want / 4, ... units, not below least, that
// alloc(units) provides; 0 if it provides none.
template <typename Alloc>
size_t alloc_most(size_t want, size_t least, Alloc alloc) {
  for (size_t n = want; n >= least && n > 0; n /= 2)
    if (alloc(n)) return n;
  return 0;
}

}  // namespace tmcs

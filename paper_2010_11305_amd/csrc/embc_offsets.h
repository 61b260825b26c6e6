// What makes offsets acceptable, for the kernels and for a host compiler.
#pragma once

#include <stdint.h>

namespace embc {

// Lookups [a, b) of a bag or a table, of L: not a range, or outside them.
constexpr bool bad_range(int64_t a, int64_t b, int64_t L) { return a < 0 || b < a || b > L; }

// The boundaries of the tables, off[t*B] for t = 0 .. T, as ranges of L lookups: true if one of
// the ranges first, first + stride, ... is bad.  When none is, the tables' positions are
// disjoint, and a workgroup that writes inside its own table's positions cannot meet
// another's, whatever the bags of the other tables look like (two tables that are valid by
// themselves may share positions when one between them runs backwards).
constexpr bool bad_boundaries(const int32_t* off, int T, int32_t B, int64_t L, int first, int stride) {
  bool bad = false;
  for (int t = first; t < T; t += stride) bad |= bad_range(off[(int64_t)t * B], off[(int64_t)(t + 1) * B], L);
  return bad;
}

}  // namespace embc

// Which of the three routes a backward call takes, by its sizes: for the runtime, and for a host
// compiler.
#pragma once

#include <stdint.h>

namespace embc {

// Small calls (k_small.hip): three launches, in which one workgroup per table sorts the table's
// lookups.  Measured steps (us), small against mid path and against the general one: 26
// tables of 2048 lookups 47, 94 and 208, 16 of 3600: 79, 102 and 230, one of 8192: 62, 92
// and 169; past 8192 lookups in a table its workgroup sorts in memory (one table of 20000:
// 159, 98 and 161).  The host knows the number of lookups of all tables together, so the
// line is drawn at 8192 per table on average and 65536 in all (nearly all of those in one
// of many tables: 0.38 ms, 0.30 on the general path before the mid path was there).
constexpr int64_t kSmallLookups = 65536;
constexpr int64_t kSmallPerTable = 8192;
constexpr int kSmallTables = 512;
constexpr int32_t kSmallBags = 65536;
constexpr bool small_call(int64_t L, int32_t B, int T) {
  return L <= kSmallLookups && L <= kSmallPerTable * T && B <= kSmallBags && T <= kSmallTables;
}

// Calls of moderate size (launch_mid_front, then as a small call): below 2M lookups, or 8M of at
// most 2^18 per table that the line below keeps.  Measured steps (us), mid against general path:
// 26 tables of 8192 lookups 125 and 247, 10 of 40000: 168 and 290, one of 2.1M in 30-lookup
// bags 306 and 468 at 16 columns, 446 and 532 at 128, 724 and 737 at 256, in one-lookup bags
// 204 and 266 (16), 355 and 420 (128); all lookups in one of 26 tables, 2M of 128 columns: 879
// and 1164.  Past 2M lookups the general path's gradient sums from LDS-staged bag blocks and
// its second stream win where a table has many lookups of wide rows: 32 tables of 250000: 694
// and 795 at 32 columns, 895 and 847 at 64, 1163 and 997 at 128, 1727 and 1345 at 256; but at
// most 2^23 columns per table (60 tables of 131000 lookups of 64 columns 870 and 1036, 64 of
// 65000 of 128: 725 and 794, 128 of 33000 of 256: 969 and 1119) or 400M in all (24 of 255000 of
// 64: 679 and 708, 12 of 255000 of 128: 539 and 557) mid is ahead.
constexpr int64_t kMidLookups = 1 << 21, kMidLookupsMost = 1 << 23, kMidPerTable = 1 << 18;
constexpr int64_t kMidColumnsPerTable = 1 << 23, kMidColumns = 3 << 27;
constexpr bool mid_call(int64_t L, int32_t B, int T, int dim) {
  if (L <= 0 || B <= 0 || T > kSmallTables) return false;
  if (L < kMidLookups) return true;
  return L < kMidLookupsMost && L <= kMidPerTable * T && (L * dim <= kMidColumnsPerTable * T || L * dim <= kMidColumns);
}

}  // namespace embc

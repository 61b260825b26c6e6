// Which of the three routes a backward call takes, and which of the two a forward call, by its
// sizes: for the launches, and for a host compiler.
#pragma once

#include <stdint.h>

namespace embc {

// Small calls (k_small.hip): three launches, in which one workgroup per table sorts the table's
// lookups.  Measured steps (us), small against mid path and against the general one: 26
// tables of 2048 lookups 44, 84 and 211, 16 of 4000: 52, 91 and 174, one of 8000: 57, 83 and
// 154, 26 of 800 ragged ones 34, 74 and 184, 8 of 3000: 46, 83 and 156.  Past 8192 lookups in a
// table its workgroup sorts in memory, and the host, which knows the number of lookups of all
// tables together, cannot see that: with nearly all of them in one of 8 tables, 16384 take
// 116 us here, 90 and 150 there, 24576: 162, 97 and 151, 65536: 374, 116 and 188; in one of 26
// tables, 24576: 164, 99 and 179, 32768: 208, 103 and 186; in one of 100, 32768: 210, 128 and 238,
// 45000: 290, 145 and 257.  So the line is drawn at 8192 per table on average, and in all where
// one table with all of them would be about as long here as on the general path (20480 and 120
// more per table: the general path's launches grow with the tables).  Calls beyond it whose
// tables hold as many lookups each lose by it (26 tables, 32768 lookups: 39 here, 78 there), but
// less than those of one long feature would on this side.  The line is 65536 where the lookups
// are a multiple of 64 bags or more: then the bags have one length, and the tables one
// number of lookups (or, once in as many calls as there are bags, they do not).
// A set is decided by one group of lanes, row by row: 8000 rows of one set take 139 us, 88 and
// 160; 12800 of one 420, 156 and 231 (one-lookup rows), of 2048 rows 191, 99 and 167; but 21440 of 16 sets
// of 3200 rows 173, 101 and 179.  Past 8192 uneven lookups in all, tables with that many rows in
// fewer than 8 sets (set_rows: of the table with the most) go to the mid path.
constexpr int64_t kSmallLookups = 65536;
constexpr int64_t kSmallPerTable = 8192;
constexpr int64_t kSmallUneven = 20480, kSmallUnevenPerTable = 120, kSmallEvenBags = 64, kSmallSetRows = 1024;
constexpr int64_t kSmallFewSets = 8;
constexpr int kSmallTables = 512;
constexpr int32_t kSmallBags = 65536;
// Rows per set of a table, as far as small_call asks for them.
constexpr int64_t small_set_rows(int64_t n_sets, int64_t rows_per_set) {
  return n_sets > 0 && n_sets < kSmallFewSets ? rows_per_set : 0;
}
constexpr bool small_call(int64_t L, int32_t B, int T, int64_t set_rows) {
  if (L > kSmallLookups || L > kSmallPerTable * T || B > kSmallBags || T > kSmallTables) return false;
  if (L <= kSmallPerTable) return true;
  const int64_t bags = (int64_t)T * B;
  if (bags >= kSmallEvenBags && L % bags == 0) return true;
  return L <= kSmallUneven + kSmallUnevenPerTable * T && set_rows <= kSmallSetRows;
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

// A forward of one kernel (k_fwd_fused) or of two, the probe and the gather.  From 2^18 lookups on the
// chip is full and two are faster.  Below (us, one kernel against two, 26 tables):
// - A row's group has few lanes to probe a long bag, the fewer the narrower the row.  16 columns: one
//   is ahead with 8 lookups per bag; 60: 37 and 34, 300: 139 and 108 (4 ways), 190 and 109 (32).
//   32 columns: up to 16 ways one is ahead or within 15% either way; 32 ways, one table of 1000
//   200-lookup bags 95 and 107, of four 750-lookup bags 276 and 219.  64 columns, 32 ways: 81 and
//   106, 225 and 209.
// - In a short bag of wide rows most lanes of a group wait for the few that probe, which matters
//   once the chip is full, and more for sets of several lines.  Up to 16 ways: 64 columns are
//   ahead throughout; 128 columns of one-lookup bags, 53000 lookups ahead, 213000: 39 and 33;
//   256 columns, 53000: 22 and 22, 213000: 66 and 54 (in 30-lookup bags 25 and 27).  From 32 ways
//   on: 64 columns, 53000 ahead, 213000: 40 and 31 (in 30-lookup bags 27 and 29); 128 columns,
//   27000 ahead, 213000: 68 and 35 (27 and 30); 256 columns, 27000: 22 and 20, 213000: 122 and 57
//   (41 and 30; 100000 in 60-lookup bags 32 and 36).
constexpr int64_t kFusedBelow = 1 << 18;
constexpr bool fused_call(int64_t L, int64_t nbags, int dim, int assoc) {
  const bool many = assoc > 16;
  const int64_t longest = dim == 16 ? 8 : dim == 32 && many ? 256 : kFusedBelow;  // lookups per bag
  if (L >= kFusedBelow || L > longest * nbags) return false;
  return many ? L * dim <= 7 << 19 || nbags * dim <= 7 << 17 : dim <= 64 || L * dim <= 3 << 22 || nbags * dim <= 1 << 21;
}

}  // namespace embc

// Sizes that scratch memory and launches are planned by (host).
#pragma once
#include <algorithm>

#include "smki_internal.h"

// ---- radix sort ----
constexpr int RS_THREADS = 256;
constexpr int RS_MAXBITS = 9;                   // digits of up to 9 bits
constexpr int RS_MAXBINS = 1 << RS_MAXBITS;
// Elements per thread: 16 (tiles of 4096) keep the tile counts, which every digit
// scans, few; up to kSmallN elements 4 (tiles of 1024), since a tile's rounds run
// one after the other and the larger tiles would leave most CUs idle: 26,000
// elements 12 us a scatter with tiles of 4096, 8 with tiles of 1024 (their counts included).
constexpr int kRounds = 16, kSmallRounds = 4;
constexpr int64_t kSmallN = int64_t(1) << 18;

// Tiles of n elements (n: the capacity where the count is on the device).
static inline int64_t radix_tiles(int64_t n) {
  return ceil_div_i64(n, RS_THREADS * (n <= kSmallN ? kSmallRounds : kRounds));
}
// What a sort of n elements writes of its scratch: the tile counts, the digit totals.
static inline size_t radix_used_bytes(int64_t n) {
  return sizeof(uint32_t) * RS_MAXBINS * (size_t)(radix_tiles(n) + 1);
}
// Scratch for a sort of any number of elements up to n.  2^18 elements make 256
// tiles and 2^18 + 1 make 65, so the most is not always at n itself: a set of
// capacity n is sorted with fewer elements where part of it is left out.
static inline size_t radix_tmp_bytes(int64_t n) {
  n = std::max<int64_t>(n, 1);
  return std::max(radix_used_bytes(n), radix_used_bytes(std::min(n, kSmallN))) + 256;
}

// ---- marks of the cells near a query ----
// Workgroups of 256 threads, eight threads a query; beyond 8,192 of them (four times
// what the card runs at once) they stride: a launch has to stay below 2^32 threads,
// which eight per query pass from 2^29 queries on.
static inline unsigned near_mark_grid(int64_t nq) {
  return (unsigned)std::min<int64_t>(ceil_div_i64(8 * nq, 256), 8192);
}

// ---- splat work units ----
#define SMKI_CHUNK 512   // most rows of one (class, block) per unit where no budget was asked for
constexpr int32_t kMostUnits = 4096;
// Units that an insert's rows are shared by, where no budget was asked for.  One
// wavefront takes a unit's rows one after the other, so a small scan whose rows lie in
// few blocks lasts as long as its longest unit (0.29 us a row at reach 3), while every
// unit adds a region to write and merge.  4,096 is 16 wavefronts on each of 256 CUs.
// Small stencils take 64 rows at a time: a quarter as many.  A block of 16^3 has regions
// of 16 to 55 KB, at most 10 on a CU: a tenth as many.  Whole call in us at 128, 256 and
// 512 rows a unit, of a street's rows in 200 to 50,000 slots:
//   reach 3, 4^3      60,000 rows 278, 300, 351;  236,000 356, 374, 424;   591,000 480, 476, 523
//   reach 3, 8^3      60,000 rows 331, 359, 393;  236,000 437, 441, 487;   591,000 542, 558, 580
//   l/res 1.5, 4^3    60,000 rows 241, 249, 258;  236,000 269, 262, 277;   591,000 312, 313, 316
//   l/res 1.5, 8^3    60,000 rows 255, 262, 277;  236,000 289, 287, 303;   591,000 396, 371, 368
//   reach 3, 16^3     60,000 rows 552, 538, 576;  236,000 890, 847, 879;   591,000 1420, 1268, 1249
//   l/res 1.5, 16^3   14,000 rows 345, 348, 364;  236,000 714, 601, 552;   591,000 1123, 838, 717
static inline int32_t unit_share(int32_t B, bool small_stencil) {
  return (B >= 16 ? 384 : kMostUnits) / (small_stencil ? 4 : 1);
}
// Units that the rows of one slot are cut into, on average: the merge of a block takes
// the units of its neighbours one after the other, and where few slots hold the rows
// there are few blocks to hide it.  The same, of a room's rows in 16 to 280 slots:
//   reach 3, 4^3      91,000 rows 269, 291, 335;  343,000 369, 351, 381
//   reach 3, 8^3      91,000 rows 334, 340, 385;  343,000 525, 435, 434
//   l/res 1.5, 4^3    91,000 rows 223, 217, 227;  343,000 321, 277, 268
//   l/res 1.5, 8^3    91,000 rows 285, 257, 255;  343,000 513, 383, 331
//   reach 3, 16^3     91,000 rows 541, 470, 484;  343,000 1347, 874, 644
// (All rows in one slot, in blocks of up to 8^3: kMostUnits whatever the stencil, as
// before the slots were counted.  7e5 rows of one class in one block of 8^3 at
// l / res = 1.5 are units of 192 rows and take 929 us; units of 512 would take 487.)
constexpr int kSlotUnits = 8;
// Rows per work unit of an insert of `rows` rows in `slots` (class, block) slots: as
// asked for at the map's creation (budget > 0), else so many that about `share` units
// share the rows and a slot has about kSlotUnits at most, in whole batches of 64,
// between 128 and SMKI_CHUNK.
// Taken on the device, in an ordinary insert and a captured one alike: a replay is cut
// into the units of the ordinary insert of its rows, whatever rows it was sized by.
__host__ __device__ static inline int32_t rows_per_unit(int32_t budget, int32_t share, int64_t rows,
                                                        int64_t slots) {
  if (budget > 0) return budget;
  const int64_t per_slot = kSlotUnits * slots;
  const int64_t units = slots <= 1 && share >= kMostUnits / 4 ? kMostUnits
                        : slots <= 1                          ? kSlotUnits
                        : per_slot < share                    ? per_slot
                                                              : share;
  const int64_t c = ((rows + units - 1) / units + SMKI_WAVE - 1) / SMKI_WAVE * SMKI_WAVE;
  return (int32_t)(c < 2 * SMKI_WAVE ? 2 * SMKI_WAVE : c > SMKI_CHUNK ? SMKI_CHUNK : c);
}
// What decides the rows per unit: the map's budget, else the share and the rows (their
// count on the device if dn_rows is set).
struct UnitRule {
  int32_t budget, share;
  int64_t rows;
  const int64_t* dn_rows;
};
// Units of at most this many rows are splatted row by row where stencils are small.
// 2e5 rows at l / res = 1.5, splat in us row by row and with lanes as rows: units of 8
// rows on average 42 and 51, of 16 rows 32 and 36 (up to 24 rows the same).
constexpr int kFewRows = 16;
// 64-lane steps that a small stencil's splat issues for `rows` rows in units of chunk:
// one a row in a unit of few rows, else per_set for each set of up to 64 rows.
__host__ __device__ static inline int64_t lane_steps(int32_t rows, int32_t chunk, int32_t per_set) {
  const int32_t full = rows / chunk, rest = rows - full * chunk;
  auto unit = [&](int32_t r) {
    return r <= kFewRows ? (int64_t)r : (int64_t)((r + SMKI_WAVE - 1) / SMKI_WAVE) * per_set;
  };
  return full * unit(chunk) + unit(rest);
}

// ---- prefix sums ----
constexpr int SCAN_THREADS = 256;
constexpr int SCAN_ITEMS = 8;
constexpr int SCAN_TILE = SCAN_THREADS * SCAN_ITEMS;
constexpr int64_t kPairTiles = 512;   // per array, for the two-launch pair scan

template <typename T>
size_t scan_tmp_elems(int64_t n) {
  size_t e = 0;
  int64_t m = n;
  while (m > SCAN_TILE) {
    m = ceil_div_i64(m, SCAN_TILE);
    e += (size_t)m + 1;
  }
  return e + 1;
}
static inline size_t scan_tmp_bytes(int64_t n) {
  return std::max<size_t>(scan_tmp_elems<int64_t>(n), 2 * kPairTiles) * sizeof(int64_t) + 256;
}

// How launches are cut: host arithmetic on sizes alone.
#pragma once

#include <stdint.h>

#include <algorithm>
#include <cmath>

#include "epicache_internal.h"

namespace epicache {

// Number of key splits of a scoring pass whose grid is `base` workgroups per split, `slots` of which the chip holds at
// once: the count (at most `most`) with the shortest estimated time.  A workgroup takes as long as its key tiles and about
// one tile's time to get going (two waves on a SIMD hide part of that from each other, and up to half a round of
// workgroups has its SIMDs to itself: 1 against 1.75).  `extra` more tiles' time per workgroup for what it repeats.
constexpr int kMostSplits = 32;
inline void pick_splits(int64_t base, int64_t slots, int tiles, double extra, int most, int* n_splits,
                        int* tiles_per_split) {
  const int cap = tiles < most ? tiles : most;
  double best = 0;
  int best_tps = tiles;
  for (int s = 1; s <= cap; s++) {
    const int tps = (tiles + s - 1) / s;
    const int eff_s = (tiles + tps - 1) / tps;
    const double rounds = (double)(base * eff_s) / (double)slots;
    const double whole = rounds <= 1 ? 1 : rounds < 4 ? (double)(int64_t)(rounds + 0.999999) : rounds + 0.5;
    const double start = (rounds <= 1 ? 1.5 : 1.0) + extra;
    const double time = (rounds <= 0.5 ? 1.0 : 1.75 * whole) * (tps + start) * (1 + 0.002 * eff_s);
    if (s == 1 || time < best) best = time, best_tps = tps;
  }
  *tiles_per_split = best_tps;
  *n_splits = (tiles + best_tps - 1) / best_tps;
}

// A fit of pass 2 with reduce = max: `each` workgroups give every CU one wave per SIMD (or as many as its LDS takes), times
// as many as `deep` of them take time[n - 1] a key tile where n share a SIMD.  Both are fitted to times: some forms leave the
// registers for more workgroups than `deep` says.
struct Residency {
  int64_t each;
  int deep;
  double time[3];
};

// Key splits of the streaming pass 2 with reduce = max, where no bit of a result depends on them (a sum over rows is added up
// in another order at the end of a split), from its times over 8 to 1024 heads of 1000 to 13000 bf16 keys of 64 to 256 bytes,
// each in 1 to 32 splits.  Three workgroups of 128 rows, or of 256 shorter ones, share a CU; a last round
// that is not full has its SIMDs to fewer waves; after four rounds they no longer end together, and the last ones wait for
// half of one.  64 heads of 64 rows, 4096 keys of 64 bytes 11.3 -> 8.0 us, 96 heads of 96 rows, 1000 keys of 192 bytes 11.1 -> 7.5,
// 896 heads of 128 rows, 4096 keys of 256 bytes 225 -> 198.
inline void pick_max_splits(const Plan& pl, int tiles, int* n_splits, int* tiles_per_split) {
  const int rows = pl.stats_rows_per_wg, nw = rows == 192 || rows == 64 ? 2 : rows == 32 ? 1 : 4;
  const bool narrow = pl.d * pl.elem < 256;
  Residency chip = {kComputeUnits * 4 / nw, 2, {1.0, 1.75, 0.0}};
  if (pl.d * pl.elem > 256) {
    if (nw < 4) chip.each = kComputeUnits * 2, chip.deep = 1;
    else chip.time[1] = 1.9;
  } else if (pl.dtype == EPICACHE_DTYPE_BF16) {
    if (rows == 128 || (rows == 256 && narrow))
      chip.deep = 3, chip.time[1] = narrow ? 1.6 : 1.75, chip.time[2] = narrow ? 2.3 : 2.6;
    else if (rows == 192 || (rows == 64 && narrow)) chip.time[1] = 1.3;
    else if (rows <= 64) chip.time[1] = 1.9;
  }
  const int64_t round = chip.each * chip.deep;
  const double full = chip.time[chip.deep - 1];
  const int cap = tiles < kMostSplits ? tiles : kMostSplits;
  double best = 0;
  int best_tps = tiles;
  for (int s = 1; s <= cap; s++) {
    const int tps = (tiles + s - 1) / s;
    const int eff_s = (tiles + tps - 1) / tps;
    const int64_t groups = (int64_t)pl.nb * pl.Hkv * eff_s, whole = groups / round, rest = groups % round;
    double rounds = (double)whole * full + (rest ? chip.time[(rest + chip.each - 1) / chip.each - 1] : 0.0);
    if (whole >= 4) rounds = ((double)groups / (double)round + 0.5) * full;
    const double time = rounds * (tps + 1.5) * (1 + 0.002 * eff_s);
    if (s == 1 || time < best) best = time, best_tps = tps;
  }
  *tiles_per_split = best_tps;
  *n_splits = (tiles + best_tps - 1) / best_tps;
}

// Where those counts are taken, by a second set of times: pass 2 of 2385 sizes, bf16 keys of 64 to 512 and fp32 keys of 288 to 512
// bytes, 8 to 896 heads of 20 to 256 rows, 1000 to 13000 keys, with the counts of pick_splits and with these.
//  - Workgroups of 128 wide rows lose: 152 of 438 sizes change and take 4 % longer on average, up to 32 % (32 heads of 96 rows,
//    13000 keys of 272 bytes 28.3 -> 37.3 us; fp32, 64 heads, 8192 keys of 288 bytes 111 -> 125).
//  - Workgroups of 32 rows of up to 64 bytes lose: 10 of 80 change, by 13 % on average (896 heads, 1000 keys 15.3 -> 18.4 us).
//  - fp32 keys of up to 256 bytes lose: both passes of 896 heads of 64 rows, 4096 keys of 256 bytes 618 -> 684 us.
//  - Of the others 450 sizes change and take 17 % less on average, up to 42 %; 4 of them take 3 to 4 % longer.
inline bool max_splits_fitted(const Plan& pl) {
  const int row_bytes = pl.d * pl.elem;
  if (row_bytes > 256) return pl.stats_rows_per_wg < 128;
  return pl.dtype == EPICACHE_DTYPE_BF16 && (pl.stats_rows_per_wg > 32 || row_bytes > 64);
}

// ---- Rows per workgroup of the scoring.  Beyond 128: 256 (4 waves x 64) or, where that pads R more, 128 (4 x 32).  192 (2 x 96) reads
// every key tile with half the waves, which pays where each CU has more than 32 tiles to get through (224 heads of
// 192 rows, 4096 keys: both passes 113 us, 122 with 256; 160 heads 87 and 89); with fewer its SIMDs are idle (128
// heads 78 and 75; 32 heads 29 and 23.5).
inline int stats_rows(const Plan& pl) {
  const auto padded = [&](int rows) { return (pl.R + rows - 1) / rows * rows; };
  const bool wide = pl.d * pl.elem > 256 || pl.dtype == EPICACHE_DTYPE_F32;  // 32 rows per wave at most
  const int64_t tiles = (int64_t)pl.nb * pl.Hkv * (padded(192) / 192) * ((pl.N + kKeyTile - 1) / kKeyTile);
  if (pl.R <= 32) return 32;
  if (pl.R <= 64) return 64;
  if (pl.R <= 128 || wide) return 128;
  if (padded(192) < padded(128) && tiles > 32 * kComputeUnits) return 192;
  return padded(128) < padded(256) ? 128 : 256;
}

// ---- The scoring workgroups of a head read the same query rows and go to one XCD.  Where the heads are no multiple of 8 that
// leaves XCDs idle or with fewer heads than others, and the workgroups go to all XCDs instead where this is more than it costs (two
// fetches of the rows, a division).  Both passes, on one XCD / on all (us, 256-byte keys):
//  - More rows than a workgroup of pass 2 holds: 1 head of 1792 rows, 16000 keys 105 / 36 (with row_groups), of 512 rows, 4000 keys
//    19.0 / 15.5; 4 heads of 512 rows, 16000 keys 38.7 / 25.4; 12 heads 70.6 / 54.0; 28 heads, 4000 keys 41.9 / 36.4.  Not with few keys: 28 heads,
//    700 keys 15.7 / 16.7; 12 heads of 1792 rows 26.1 / 27.7; 4 heads of 512 13.6 / 14.1.
//  - Otherwise a head has 32 key splits at most, one per CU of an XCD, and only an XCD with more heads than others takes longer: 12 heads of
//    192 rows, 4000 keys 21.0 / 16.4, 16000 keys 45.0 / 32.3; 28 heads, 4000 keys 30.6 / 23.1; but of 64 rows 14.5 / 15.4.
// The fullest XCD has to have an eighth more heads than the average: with 44 heads of 256 rows, 864 keys the step took 24.0 / 25.0, with 22 of
// 256 rows, 7729 keys of 128 bytes 56.9 / 58.2.
inline bool spreads_heads(const Plan& pl) {
  const int64_t heads = (int64_t)pl.nb * pl.Hkv;
  if (pl.N < 2000 || heads > (heads + 7) / 8 * 7) return false;
  return pl.R > pl.stats_rows_per_wg || (heads > 8 && heads * pl.R * pl.N >= 8000000);
}

// ---- Groups of the four waves of pass 2 that share out the query rows where those are more than one workgroup's (score_reduce, bf16
// keys of 64 or 128 elements): as many as leave the head's XCD, or the chip, one round of workgroups of 256 / groups keys, and a workgroup
// 160 KB of LDS.  Both passes in 1 / 2 / 4 groups (us): 8 heads of 1792 rows, 700 keys 34.9 / 26.6 / 22.0, 4000 keys 46.6 / 38.7 / 49.0;
// of 512 rows, 700 keys 17.4 / 15.2 / 13.8, 4000 keys 19.5 / 17.4 / 22.6, 16000 keys 39 / 46 / 80.
inline int row_groups(const Plan& pl) {
  const int64_t heads = (int64_t)pl.nb * pl.Hkv;
  for (int groups = 4; groups >= 2; groups /= 2) {
    const int64_t blocks = (pl.N + 256 / groups - 1) / (256 / groups);
    const int64_t lds = groups * 2 * 64 * (pl.d * pl.elem) + (int64_t)pl.Rpad * 4;
    const bool one_round = pl.spread ? heads * blocks <= kComputeUnits : (heads + 7) / 8 * blocks <= kComputeUnits / 8;
    if (one_round && lds <= 160 * 1024) return groups;
  }
  return 1;
}

// ---- Selection and compaction in one launch (launch_select_compact).
// 1024 threads for more than 2048 scores: the selection of 2048 in 512 threads 12.4 us, in 1024 12.9; of 4096 18.5 and 17.9.
inline int select_compact_threads(int n_scored) { return n_scored <= 2048 ? 512 : 1024; }

// Every (head, tensor) selects for itself, so K and V do it twice.  That is lost in a CU that has nothing else to do, and behind
// a copy that is long enough; where neither holds, the launch takes longer than topk_select + compact_rows.  Whole steps in
// two launches / one (us): 128 heads of 16384 scores, 128 rows of 16 bytes kept 63.5 / 58.3; of 4096, 1000 rows of 16 36.8 /
// 33.8.  384 heads of 2048, 128 rows of 16 35.8 / 34.8; 512 heads of 1024, 256 rows of 16 33.9 / 34.0, of 32 37.2 / 34.6; 1024
// heads of 300, 128 rows of 16 33.0 / 36.1.  160 heads of 4096, 1000 rows of 16 44.0 / 46.8, of 64 50.4 / 47.8; 512 heads of
// 4096, 256 rows of 16 62.4 / 76.9, of 64 69.4 / 77.9, of 256 234 / 238, 1000 rows of 128 147 / 144; 160 heads of 16384, 1500
// rows of 64 96 / 101, of 128 168 / 159.  (192 heads of 4096, 2000 rows of 64, on the wrong side: 63.3 / 65.5.)
inline bool select_compact_pays(int64_t problems, int n_scored, int64_t kept_bytes) {
  if (problems <= kComputeUnits) return true;
  return kept_bytes >= (n_scored <= 2048 ? 8 << 10 : std::max<int64_t>(64 << 10, 8 * (int64_t)n_scored));
}

// Ranges that the kept rows of a (head, tensor) are cut into, or 0 where the launch is not taken.  problems: heads times 2.
//
// Up to 64 MB of kept rows, 256 KB for every CU; beyond, the copy is what counts, and the slices of compact_rows are as good.
// Kernel times, rows of 256 bytes, topk_select + compact_rows / this one: 32 heads, 512 of 1024 rows kept 10.2 / 9.8 us, 2048
// of 4096 22.0 / 18.3, 4096 of 8192 42.0 / 30.2; 24 heads, 3000 of 4336 27.6 / 21.3; 12 heads, 6000 of 9000 42 / 24.6; 64
// heads, 2048 of 4096 31.1 / 28.2; 8 heads, 8192 of 16384 47.5 / 24.5.
// As many ranges as give the busiest CU the shortest way: its workgroups times their rows, and for each of them the time of
// 40 KB for the selection (it takes 1.7 us of 4096 scores where a CU has one workgroup, 5 where it has two).
inline int select_compact_parts(int64_t problems, int n_scored, int n_total, int row_bytes) {
  if (n_scored > 16384 || problems * n_total * row_bytes > (64 << 20)) return 0;
  if (!select_compact_pays(problems, n_scored, (int64_t)n_total * row_bytes)) return 0;
  const int per_round = select_compact_threads(n_scored) / (row_bytes / 16);  // rows
  const int least = (n_total + 16 * per_round - 1) / (16 * per_round), most = std::max(least, std::min(32, n_total / 64));
  int parts = 0;
  int64_t best = INT64_MAX;
  for (int p = least; p <= most && p <= 32; p++) {
    const int64_t way = ((problems * p + kComputeUnits - 1) / kComputeUnits) * ((n_total + p - 1) / p + 40 * 1024 / row_bytes);
    if (way < best) best = way, parts = p;
  }
  return parts;
}

// The ranges of a (head, tensor) go to one XCD, whose L2 has the scores once, unless some XCD would then have more workgroups than CUs
// while the chip has enough: two of them on a CU select one after the other.  Steps in one XCD / all (us), 4000 of 9000 rows of 256
// bytes: 3 heads 24.3 / 24.6, 5 36.5 / 25.9, 7 36.1 / 26.7, 9 36.3 / 28.3, 13 39.5 / 31.1, 20 36.4 / 36.4; 1 head, 13000 of 14000
// 26.4 / 28.0; 5 heads, 1000 of 2000 12.6 / 13.9.
inline bool spreads_ranges(int64_t problems, int parts) {
  return (problems + 7) / 8 * parts > kComputeUnits / 8 && problems * parts <= kComputeUnits;
}

// ---- Slices of whole 64-byte parts of a row in compact_rows, each a workgroup's, until every CU has one (256 of them).  Slices
// that end inside 64 bytes, or more of them than that, cost more than they bring: 64 heads of 96-element rows 12.4 us in one slice, 15.8
// in two of 96 bytes; 896 heads 338 us in one slice, 347 in two, 453 in four.
inline int row_slices(int64_t problems, int row_bytes) {
  int slices = 1;
  while (problems * slices < kComputeUnits && row_bytes / 16 % (slices * 8) == 0) slices *= 2;
  return slices;
}

// ---- Ranges that the kept rows of a (head, tensor) are cut into by compact_ranges, or 0 where compact_rows moves them.
// problems: heads times 2.  Whole steps with compact_rows / compact_ranges (us), rows of 256 bytes unless given:
//  - Few heads leave compact_rows with a workgroup per 64-byte slice: 2 heads, 11000 of 18000 rows 61 / 35; 8 heads 76 / 45, 8 of
//    30000 of 40000 rows 217 / 131; 16 heads, 13000 of 14000 92 / 67; 32 heads, 8000 of 20000 rows of 128 bytes 73 / 55; 48 heads, 3000
//    of 17000 rows of 192 bytes 74.5 / 63.9.  The ranges' start and their claims take one or two us, and longer behind a ragged selection, so the way
//    of a workgroup of compact_rows, which has one slice of all rows, has to be as long: 48 KB (ragged 96), or 16 (32) where all heads' rows are
//    1 MB (4 MB) or more, which is more than a CU's share of them.  Over 3801 uniform and 13336 ragged steps of 1 to 63 heads, 48 to 1500 KB a head, rows of 64 to 512
//    bytes that is 0.1 and 0.2 % behind the faster of both on average (by the bytes of a head alone, from 288 KB on, 2.2 and 1.2 %).
//    40 ragged heads, 1631 rows of 128 56.0 / 53.0; 18 heads, 227 of 539 21.9 / 23.0; 48 heads, 312 of 561 22.6 / 23.5; 4 heads, 590 of 1014 rows of 192
//    18.1 / 19.2.  (On the wrong side: 60 ragged heads, 414 of 480 22.0 / 24.0.)
//  - Beyond 448 problems a range is a load of its workgroup without another chunk behind it: 896 heads, 2048 of 4096 rows
//    516 / 493, 7000 of 9000 1644 / 1528; 256 heads, 13000 of 14000 810 / 751; 448 heads, 2500 of 3000 rows of 512 bytes 578 / 526; 300 of 600
//    rows 45.2 / 44.3, 4000 of 6000 rows of 16 bytes 75.0 / 73.9; not with few short chunks (448 heads, 128 of 300 rows 25.3 / 25.7).
//  - In between compact_rows has one or two workgroups per CU, and only long ways are shorter in ranges: 112 heads, 7000 of 9000 rows 200 / 186,
//    224 heads 399 / 371, but 112 heads, 2000 of 3000 rows of 192 bytes 54.4 / 55.5, 19000 of 20000 rows of 32 bytes 93 / 97.5;
//    96 heads, 10000 rows of 16 bytes 57.4 / 63.6.  (64 heads, 2500 of 3000 rows of 512 bytes, on the wrong side: 82.5 / 83.7.)
// Where the chip has more than two of them per CU, ranges of eight rounds of a workgroup, two of which share a CU; else as many as give
// the busiest CU the shortest way, of up to sixteen rounds: its workgroups times their rows, and for each of them the time of 16 KB.
// longest: the most rows of a head, whose chunks are the way in compact_rows.
inline int compact_parts(int64_t problems, int n_keep, int row_bytes, int longest, bool ragged) {
  const int64_t bytes = (int64_t)n_keep * row_bytes, way_kb = bytes / row_slices(problems, row_bytes) >> 10;
  const int64_t all_mb = problems / 2 * bytes >> 20;
  if (problems >= 128 ? bytes < (48 << 10) : way_kb < (ragged ? 96 : 48) && (way_kb < (ragged ? 32 : 16) || all_mb < (ragged ? 4 : 1))) return 0;
  if (problems >= 128 && problems <= 448 && (int64_t)longest * row_bytes < (1 << 20)) return 0;
  const int eight = 8 * (1024 / (row_bytes / 16));  // rows
  const int full = (n_keep + eight - 1) / eight, least = (full + 1) / 2;
  if (least > 32) return 0;  // one report bit each
  if (problems * full > 2 * kComputeUnits && full <= 32) return full;
  int parts = 0;
  int64_t best = INT64_MAX;
  for (int p = least; p <= 32; p++) {
    const int64_t way = ((problems * p + kComputeUnits - 1) / kComputeUnits) * ((n_keep + p - 1) / p + 16 * 1024 / row_bytes);
    if (way < best) best = way, parts = p;
  }
  return parts;
}
// The ranges of heads that keep n_keep rows on average, or in a ragged batch up to `most`: as for n_keep, and more of the same rows behind
// them, whose workgroups leave at once where a head has not so many.  Where one holds the average head, or the chip has more than two
// per CU, they are as long as eight rounds take.  Cut for the longest head instead, every head's rows went to as many workgroups: pooled
// selection over 276 heads of 8 an item, 319 of 2059 rows of 128 bytes, whole step 578 us (compact_rows 513), 464 heads, 919 of 1025 rows of 256
// 134 (121, now 124), 240 heads, 205 of 341 34.1 in two ranges of the average (32.1 in one).
struct CompactRanges {
  int parts, rows;
};
inline CompactRanges compact_ranges_of(int64_t problems, int n_keep, int most, int row_bytes, bool ragged) {
  const int parts = compact_parts(problems, n_keep, row_bytes, most, ragged), longest = 1024 / (row_bytes / 16) * 16;
  if (parts == 0) return {0, 0};
  int rows = (n_keep + parts - 1) / parts;
  if (most <= n_keep) return {parts, rows};
  if (parts == 1 || problems * parts > 2 * kComputeUnits) rows = longest / 2;
  rows = std::max(rows, (most + 31) / 32);  // one report bit each
  if (rows > longest) return {0, 0};
  return {(most + rows - 1) / rows, rows};
}
// Whether they pay also behind a launch that clears the claims, which makes a call 1.2 to 2.9 us longer (5 us by itself).
// epicache_compact in compact_rows / in both launches (us, rows of 256 bytes unless given):
//  - Few heads: the two launches take 11 us, compact_rows 8 where it has one chunk of 2048 rows and more by the heads: 2 heads,
//    2048 of 2560 rows 7.9 / 11.0, 3072 of 7680 9.8 / 10.9, 4096 of 5120 11.9 / 11.0; 8 heads, 2048 8.2 / 11.2, 3072 12.7 / 10.7; 16
//    heads, 1536 9.0 / 10.9, 2048 11.5 / 10.7; 32 heads, 1536 10.9 / 11.2, 2048 14.7 / 13.4; rows of 512 bytes, 32 heads, 1024 12.2 /
//    13.3; 63 heads 27.3 / 25.3.  (On the wrong side: 1 head, 4096 of 5120 8.7 / 11.2; 8 heads,
//    3072 of 5222 rows of 128 9.5 / 11.0, 2048 of 3481 of 512 12.5 / 10.8.)
//  - Many heads: 401 heads, 184 KB 59.5 / 57.8, 440 heads, 284 KB 100.7 / 95.8, 593 heads, 315 KB 150.9 / 141.4, 896 heads, 512 KB 339 / 315.  Where
//    few rows move, with KeyDiff scoring and selection: 372 heads, 1145 of 1373 81.7 / 86.0, 768 heads, 700 of 1200 113.8 / 120.3, 640 heads,
//    1500 of 2300 206.1 / 203.6: from 320 KB a head and 256 MB on.
//  - One range a head needs no claims, and no launch for them: 896 heads, 342 of 1606, the same calls 139.7 / 136.0.
inline bool compact_parts_pay_for_claims(int64_t problems, int n_keep, int row_bytes, int parts) {
  const int64_t bytes = (int64_t)n_keep * row_bytes;
  if (problems >= 128) return problems * bytes >= (parts == 1 ? (int64_t)128 << 20 : std::max((int64_t)256 << 20, problems * (320 << 10)));
  return bytes >= (384 << 10) && n_keep >= (problems <= 8 ? 4096 : problems <= 16 ? 3072 : problems <= 64 ? 2048 : 0);
}

// ---- Workgroups of patch_attention_mfma: eight waves as row_waves blocks of 32 query rows times `groups` groups of waves that
// take every groups-th tile of keys, and key_splits workgroups of split_keys keys each (the last has what is left) for the same rows.
struct AttentionShape {
  int row_waves, groups, key_splits, split_keys;
};
inline int attention_blocks(const Plan& pl) { return (pl.R + 31) / 32; }
// Floats that a row of one key split leaves for merge_attention: its output, reference and sum.
inline int64_t attention_record(const Plan& pl) { return pl.d + 2; }

// The shape with the shortest estimated time.  Estimate: rounds of workgroups (one per CU) on the fullest XCD times (a wave's keys and
// a start), what the workgroups read of K and V from L2, and for key splits a launch more and the records.  Fitted per row layout
// to the times of 113 sizes (2 to 416 heads of 32 to 1792 rows, 450 to 18000 keys of 32, 64, 96 and 128 elements) and, for the fullest XCD
// and rows of up to 32 elements, of 409 more (1 to 400 heads of 16 to 1792 rows, 300 to 18000 keys), each in all shapes with up to three rounds of
// workgroups.  Checked on 479 others: the attention by keys per wave alone / by this / in the best shape, geometric means (us) without
// room: 128 elements 46.5 / 42.3 / 42.8, 96 38.4 / 34.4 / 34.9, 64 33.1 / 31.8 / 31.8, 32 31.3 / 29.4 / 29.8; with it, this / best: 34.6 / 34.0, 28.9 /
// 28.8, 28.7 / 28.1, 27.0 / 26.2; two of them 8 and 15 % longer than by keys per wave (248 heads of 128 rows, 3108 keys of 64 59.6 / 64.1; 32 of
// 200, 10711 of 64 54.1 / 62.1).  By rounds of the whole chip 7 of 409 took 1.6 to 1.75 times as long (36 heads of 224 rows, 1505 keys 36.1 us
// where five heads meet on an XCD of 32 CUs, 20.9 with four workgroups a head).  More than 32 splits: 2 heads of 50 rows, 2866
// keys 24.7 us in 45, 17.3 in 32; 1 head of 64, 2743 keys of 64 22.3 in 44, 15.4 in none.  The attention of 8 heads of 192 rows,
// 12008 keys of 128 elements: 140 us in 48 workgroups, 19 in 16 splits of 8 times two.
// `room`: the caller has room for what the key splits leave.
inline AttentionShape attention_shape(const Plan& pl, bool room) {
  struct Times {
    double thousand_keys[4], start, merge, record;  // us; [row_waves = 8, 4, 2, 1]; per row and split
  };
  const bool whole_parts = pl.d == 128;  // one product with V per weight; otherwise three (patch_attn.hip)
  const Times t = whole_parts  ? Times{{19.7, 23.5, 30.4, 19.6}, 5, 3.3, 1.2e-4}
                  : pl.d > 64  ? Times{{29.5, 35.5, 41.0, 29.0}, 3, 5, 1.7e-6 * pl.d}
                  : pl.d > 32  ? Times{{20.5, 27.0, 31.0, 29.0}, 3, 5, 1.7e-6 * pl.d}
                               : Times{{23.0, 20.0, 29.0, 26.0}, 3, 5, 1.7e-6 * pl.d};
  const int most_groups = pl.d <= 64 ? 8 : 4;  // what fits 160 KB of LDS
  const int64_t heads = (int64_t)pl.nb * pl.Hkv;
  const int blocks = attention_blocks(pl), keys = pl.N + (pl.causal_patch ? pl.p : 0), tiles = (keys + 63) / 64;
  AttentionShape shape = {8, 1, 1, keys};
  double best = 0;
  for (int i = 0, w = 8; w >= 1; w /= 2, i++) {
    const int groups = std::min(8 / w, most_groups);
    const int64_t row_groups = (blocks + w - 1) / w, per_split = heads * row_groups;
    auto consider = [&](int splits, int each) {
      // those of a head and split go to one XCD
      const double rounds = (double)((heads * splits + 7) / 8 * row_groups) / (kComputeUnits / 8);
      double time = (rounds < 4 ? std::ceil(rounds) : rounds + 0.5) * (t.thousand_keys[i] * 1e-3 * each / groups + t.start);
      time += 0.02e-6 * (double)(per_split * splits) * each * pl.d;
      // the errors of the estimate are no reason for a split: 22 heads of 256 rows, 7729 keys of 64 elements are estimated alike
      // and the step takes 56.7 us without, 57.6 with splits
      if (splits > 1) time = 1.05 * (time + t.merge + t.record * (double)(heads * pl.R * splits));
      if (best == 0 || time < best) best = time, shape = {w, groups, splits, each};
    };
    consider(1, keys);
    if (!room) continue;
    for (int halves : {1, 2, 4, 6}) {  // as many splits as half a round of workgroups has, one, two, three
      const int most = (int)std::min<int64_t>(halves * kComputeUnits / 2 / per_split, std::min(tiles, 32));
      if (most < 2) continue;
      const int each = (tiles + most - 1) / most;
      if (each < tiles) consider((tiles + each - 1) / each, 64 * each);
    }
  }
  return shape;
}
// Bytes that the key splits leave.
inline size_t attention_room(const Plan& pl) {
  if (pl.dtype != EPICACHE_DTYPE_BF16 || pl.d > 128) return 0;
  const AttentionShape shape = attention_shape(pl, true);
  if (shape.key_splits == 1) return 0;
  return (size_t)pl.nb * pl.Hkv * shape.key_splits * pl.R * attention_record(pl) * sizeof(float);
}

// ---- Centroids that a wave of match_queries takes at a time: three instead of two where that makes fewer rounds, each a chain
// of loads and lane sums (1 query, 10 episodes of 4096 dims 5.3 us instead of 7.4).  Places that hold no episode read the last
// one again: with as many rounds as two they are what a call takes longer (1000 queries, 16 episodes of 4096 dims 16.9 us with
// two, 20.7 with three; 4 of 1024 4.5 and 5.0).  Beyond two queries per CU the reads count more than the rounds (1000 queries, 17
// episodes of 1024 dims 7.6 and 8.1 us, 25 of 1536 12.2 and 11.5).
constexpr int kMatchWaves = 4;
inline int match_rows(int n_queries, int n_episodes) {
  auto rounds = [&](int rows, int wave) {
    return (n_episodes - wave + rows * kMatchWaves - 1) / (rows * kMatchWaves);
  };
  const bool fewer_rounds = rounds(3, 0) < rounds(2, 0);
  if (n_queries <= 2 * kComputeUnits) return fewer_rounds ? 3 : 2;
  int reads2 = 0, reads3 = 0;
  for (int wave = 0; wave < kMatchWaves; wave++) reads2 += 2 * rounds(2, wave), reads3 += 3 * rounds(3, wave);
  return reads3 < reads2 || (fewer_rounds && (rounds(3, 0) == 1 || reads3 <= reads2 + 1)) ? 3 : 2;
}

// ---- Workgroups of episode_medoids: for each cluster of up to 256, as many of 16 waves with four rows each as its share of the
// segments has 64 rows for, and no more than one per CU in all (both calls of 24 clusters of 4000 segments, 384 dims, 22.5 ->
// 17.9 us against four waves with three rows).  With more clusters every CU has several workgroups, and four waves list a
// cluster's few members in less time than sixteen (300 clusters of 30 segments, 384 dims, 40.0 and 45.1 us; 1000 of 8, 100
// dims, 29.9 and 42.4).  Rows of more than 2048 dims are better dealt to more workgroups of four waves (10 clusters of 64
// segments, 4096 dims, 25.1 and 29.2; 24 of 1000 170 and 179), though clusters of two take up to 30 % longer so.
struct MedoidShape {
  int threads, per_cluster;
};
inline MedoidShape medoid_shape(int n_segments, int n_clusters, int dim) {
  const bool large = n_clusters <= kComputeUnits && dim <= 2048;
  const int64_t each = large ? 64 : 12, most = kComputeUnits / n_clusters;
  const int64_t wanted = large ? (n_segments + each * n_clusters - 1) / (each * n_clusters) : n_segments / (each * n_clusters);
  return {large ? 1024 : 256, (int)std::max<int64_t>(1, std::min(most, wanted))};
}

}  // namespace epicache

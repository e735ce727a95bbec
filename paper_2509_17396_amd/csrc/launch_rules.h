// How launches are cut: host arithmetic on sizes alone.
#pragma once

#include <stdint.h>

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
    if (rows == 128 || (rows == 256 && narrow)) chip.deep = 3, chip.time[1] = narrow ? 1.6 : 1.75, chip.time[2] = narrow ? 2.3 : 2.6;
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

}  // namespace epicache

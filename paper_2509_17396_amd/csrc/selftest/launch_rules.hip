// The rules of launch_rules.h, for the tests.  Not part of the library; host code only.
#include <string.h>

#include "../launch_rules.h"

#define EXPORT extern "C" __attribute__((visibility("default")))

// 1 where pass 2 with reduce = max takes its key splits from the fit, with the counts of both estimates
EXPORT int max_splits(int dtype, int d, int rows_per_wg, int heads, int tiles, int* fitted, int* estimated) {
  epicache::Plan pl;
  memset(&pl, 0, sizeof(pl));
  pl.nb = 1, pl.Hkv = heads, pl.d = d, pl.dtype = dtype, pl.elem = dtype == EPICACHE_DTYPE_F32 ? 4 : 2;
  pl.stats_rows_per_wg = rows_per_wg;
  const int waves = rows_per_wg == 192 || rows_per_wg == 64 ? 2 : rows_per_wg == 32 ? 1 : 4;
  const int fit = d * pl.elem > 256 && waves < 4 ? 2 : 8 / waves;
  int tiles_per_split;
  epicache::pick_max_splits(pl, tiles, fitted, &tiles_per_split);
  epicache::pick_splits(heads, epicache::kComputeUnits * fit, tiles, 0.5, epicache::kMostSplits, estimated, &tiles_per_split);
  return epicache::max_splits_fitted(pl);
}

EXPORT int select_compact_parts(int heads, int n_scored, int n_total, int row_bytes) {
  return epicache::select_compact_parts(2 * (int64_t)heads, n_scored, n_total, row_bytes);
}

EXPORT int match_rows(int n_queries, int n_episodes) { return epicache::match_rows(n_queries, n_episodes); }

EXPORT int medoid_shape(int n_segments, int n_clusters, int dim, int* per_cluster) {
  const epicache::MedoidShape s = epicache::medoid_shape(n_segments, n_clusters, dim);
  *per_cluster = s.per_cluster;
  return s.threads;
}

// Whether the scoring's workgroups go to all XCDs; *groups: of the waves of the key-stationary pass 2, 0 where it streams the keys or has none
EXPORT int score_form(int dtype, int heads, int rows, int n, int d, int* groups) {
  epicache::Plan pl;
  memset(&pl, 0, sizeof(pl));
  pl.nb = 1, pl.Hkv = heads, pl.R = rows, pl.Rpad = (rows + 63) / 64 * 64, pl.N = n, pl.d = d, pl.dtype = dtype;
  pl.elem = dtype == EPICACHE_DTYPE_F32 ? 4 : 2;
  pl.stats_rows_per_wg = epicache::stats_rows(pl);
  pl.spread = epicache::spreads_heads(pl);
  const bool folded = dtype == EPICACHE_DTYPE_BF16 && (d == 64 || d == 128);
  *groups = pl.R <= pl.stats_rows_per_wg ? 0 : folded ? epicache::row_groups(pl) : 1;
  return pl.spread;
}

EXPORT int spreads_ranges(int heads, int parts) { return epicache::spreads_ranges(2 * (int64_t)heads, parts); }

static epicache::Plan attention_plan(int heads, int rows, int patch, int n, int causal, int d) {
  epicache::Plan pl;
  memset(&pl, 0, sizeof(pl));
  pl.nb = 1, pl.Hkv = heads, pl.R = rows, pl.p = patch, pl.N = n, pl.causal_patch = causal, pl.d = d;
  pl.dtype = EPICACHE_DTYPE_BF16, pl.elem = 2;
  return pl;
}

// Row blocks of a workgroup of patch_attention_mfma without room for key splits
EXPORT int attention_row_waves(int heads, int rows, int n, int d) {
  return epicache::attention_shape(attention_plan(heads, rows, rows, n, 0, d), false).row_waves;
}

// The workgroups of patch_attention_mfma with room for key splits: {row_waves, groups, key_splits, split_keys}; the bytes of that room
EXPORT int64_t attention_shape(int heads, int rows, int patch, int n, int causal, int d, int* out) {
  const epicache::Plan pl = attention_plan(heads, rows, patch, n, causal, d);
  const epicache::AttentionShape s = epicache::attention_shape(pl, true);
  out[0] = s.row_waves, out[1] = s.groups, out[2] = s.key_splits, out[3] = s.split_keys;
  return (int64_t)epicache::attention_room(pl);
}

EXPORT int compact_parts(int heads, int n_keep, int row_bytes) {
  return epicache::compact_ranges_of(2 * (int64_t)heads, n_keep, n_keep, row_bytes, false).parts;
}

// The same of a ragged batch whose heads keep up to `most` rows
EXPORT int compact_ranges(int heads, int n_keep, int most, int row_bytes, int* rows) {
  const epicache::CompactRanges r = epicache::compact_ranges_of(2 * (int64_t)heads, n_keep, most, row_bytes, true);
  *rows = r.rows;
  return r.parts;
}

EXPORT int compact_parts_pay_for_claims(int heads, int n_keep, int row_bytes) {
  const int parts = epicache::compact_ranges_of(2 * (int64_t)heads, n_keep, n_keep, row_bytes, false).parts;
  return epicache::compact_parts_pay_for_claims(2 * (int64_t)heads, n_keep, row_bytes, parts);
}

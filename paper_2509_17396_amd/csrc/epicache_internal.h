// Internal declarations shared by the HIP translation units of libepicache.
// Not part of the C ABI (see include/epicache.h).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "epicache.h"

namespace epicache {

// Everything the launchers need, derived once on the host from epicache_params.
struct Plan {
  int nb, Hq, Hkv, G, d, p;
  int N;        // context rows scored: n_cached + n_block
  int R;        // rows that vote for one KV head: G * p
  int Rpad;     // R rounded up to 64
  int M;        // budget
  int n_keep;   // min(M, N)
  int dtype, reduce;
  int causal_patch;  // the p rows after a head's context are the patch's keys, seen causally by the queries
  int elem;     // bytes per element of Q/K/V
  uint32_t heads_magic;  // bh / Hkv and row / p in the kernels without a division: ceil(2^32 / Hkv) ...
  float inv_p;           // ... and 1 / p
  float c2;     // softmax scale * log2(e): logits are handled in base 2
  int64_t qsb, qsh, qst, ksb, ksh, kst;  // strides in elements
  // score kernels
  int use_mfma;     // MFMA path (rows of at most 512 bytes), else the generic fp32 path
  int stats_rows_per_wg;  // query rows per workgroup of the row-statistics pass
  int n_splits;     // key splits of the row-statistics pass
  int live_splits;  // set for the reduction: how many of a row's split records count (1 once they are combined)
  int tiles_per_split;
  int reduce_splits;  // key splits of the streaming reduction pass
  int reduce_tiles_per_split;
  int spread;       // the workgroups of a head go to all XCDs (spreads_heads in launch_rules.h)
  // workspace layout (byte offsets, 256-aligned)
  size_t off_stats, off_scores, off_keep, off_lse, ws_total;
  uint32_t* claims;   // null, or what the reduction pass sets to 0: kClaimsPerHead per (b, h)
  // ragged batches: device arrays indexed by b * Hkv + h, null in the uniform calls
  const int32_t* n_ctx;   // context rows per (b, h), at most N; N is then the pitch of a score row
  const int32_t* n_kept;  // rows kept per (b, h), read by the compaction
  int keep_stride;        // pitch of a row of kept indices (n_keep in the uniform calls)
  size_t off_select;      // per-(b, h) threshold records of the ragged selection
};

// Claims of a (b, h): for K and for V the number of parts taken, and a bit per part whose rows are all in registers.  K and V
// in a 128-byte line of their own: packed, the atomics of all heads met on a few lines (32 heads of 8 parts: 27 us, 21).
constexpr int kClaimPitch = 16, kClaimsPerHead = 4 * kClaimPitch;

// Context rows of (b, h): the per-head length of a ragged batch, clamped to what the strides were checked for.
__device__ __forceinline__ int ctx_rows(const Plan& pl, int bh) {
  if (!pl.n_ctx) return pl.N;
  const int n = pl.n_ctx[bh];
  return n < 0 ? 0 : (n > pl.N ? pl.N : n);
}

// bh / Hkv for bh < 65536 (the error of the reciprocal, below Hkv / 2^32, times bh stays below 1 / Hkv).
__device__ __forceinline__ int batch_of(const Plan& pl, int bh) {
  return pl.Hkv == 1 ? bh : (int)__umulhi((uint32_t)bh, pl.heads_magic);
}
// Query head within the group and patch token of scoring row r: r / p and r % p.  r <= 2^14 + 255, so the quotient's
// distance from the next integer, at least 0.5 / p, is more than its rounding error.
__device__ __forceinline__ void head_and_token(int p, float inv_p, int r, int& g, int& t) {
  g = (int)(((float)r + 0.5f) * inv_p);
  t = r - g * p;
}

// Compute units of the one target of this build, MI355X (gfx950): 8 XCDs x 32.  It steers how a launch is cut, no result.
constexpr int kComputeUnits = 256;
constexpr int kKeyTile = 64;     // keys staged per LDS tile in the statistics pass

// By one thread each: the claims of (b, h) before the first workgroup of launch_select_compact or launch_compact looks at them.
__device__ __forceinline__ void clear_claims(const Plan& pl, int bh, bool first_of_head) {
  if (pl.claims && first_of_head && threadIdx.x < 4) pl.claims[(size_t)bh * kClaimsPerHead + threadIdx.x * kClaimPitch] = 0;
}

// Each launcher enqueues on `stream` and returns a hipError_t.
// `stats_ready`: the row statistics are already in `stats` (one split); only the reduction pass runs.
hipError_t launch_score_generic(const Plan& pl, const void* q, const void* k, float* scores,
                                float2* stats, bool stats_ready, hipStream_t stream);
// row_lse: null, or the caller's natural-log normalisers [nb, Hq, p]; then only the reduction pass runs.
hipError_t launch_score_mfma(const Plan& pl, const void* q, const void* k, float* scores, float2* stats,
                             const float* row_lse, hipStream_t stream);
// Room for the claims in `stats`, beside what the reduction pass of that launch reads there.  with_lse: row_lse is not null.
uint32_t* claims_in_stats(const Plan& pl, float2* stats, bool with_lse);
hipError_t launch_lse_to_stats(const Plan& pl, const float* row_lse, float2* stats, hipStream_t stream);
// appended: the rows N .. N + appended - 1 are kept whatever they score, behind the n_keep selected ones
hipError_t launch_topk(const Plan& pl, const float* scores, int32_t* keep, int appended, hipStream_t stream);
hipError_t launch_iota_keep(const Plan& pl, int32_t* keep, hipStream_t stream);
// dst = reduce(dst, src) elementwise over [nb, Hkv, N] scores (pl.reduce)
hipError_t launch_combine_scores(const Plan& pl, float* dst, const float* src, hipStream_t stream);
// pl.claims: null, or cleared ones that no other launch has used (not read where the rows of a head are one range).
// beside_scoring: the launch runs next to scoring kernels on another stream and has to fit between their waves
hipError_t launch_compact(const Plan& pl, const int32_t* keep, void* k, void* v, bool beside_scoring,
                          hipStream_t stream);
// All claims of `heads` heads, kClaimsPerHead each.
hipError_t launch_clear_claims(uint32_t* claims, int heads, hipStream_t stream);
// Selection and compaction in one launch, for steps that are too small to fill the chip with either: `scored` is the plan
// of the scores (N, n_keep, claims), `cache` that of the rows that are moved.  keep_opt: null, or where the kept indices go
// (rows of cache.keep_stride).  *done: whether the launch took the step; if not, launch_topk and launch_compact do.
// patience: how often a workgroup looks whether the ranges below its own are loaded.  They are within a few microseconds of
// its own; a look takes 0.14 us with the chip to itself, all of them 0.14 s.
constexpr int kClaimPatience = 1 << 20;
hipError_t launch_select_compact(const Plan& scored, const Plan& cache, const float* scores, int32_t* keep_opt, int appended,
                                 void* k, void* v, hipStream_t stream, bool* done, int patience = kClaimPatience);
size_t select_ragged_record_bytes(const Plan& pl);
// KeyDiff scoring: chunk sums of the keys live at the start of the workspace.
size_t keydiff_workspace_bytes(const Plan& pl);
// patience: how often a workgroup of the one-pass form looks whether the others of its head have arrived before it
// does without them.  With the chip to itself a call's workgroups all arrive within 32 looks (896 heads of 4096 rows, 1024
// of 16384); doing without costs 0.1 ms (4096 rows) to 0.4 ms (32768), about as long as 512 looks.
constexpr int kKeydiffPatience = 512;
hipError_t launch_score_keydiff(const Plan& pl, const void* k, float* scores, void* workspace, hipStream_t stream,
                                int patience = kKeydiffPatience);
// Ragged selection: per-(b, h) (select == per head) or per-b pooled thresholds, then the kept indices.
hipError_t launch_select_ragged(const Plan& pl, int select, const float* scores, const int32_t* budgets,
                                int32_t* keep, int32_t* n_kept, void* records, hipStream_t stream);

// Attention output and log-sum-exp of the patch queries (dense out [nb, Hq, p, d], lse [nb, Hq, p]).
// room_opt: null, or attention_room(pl) bytes that let several workgroups share the keys of a row.
hipError_t launch_patch_attention(const Plan& pl, const void* q, const void* k, const void* v, void* out,
                                  float* lse, float* room_opt, hipStream_t stream);
// Episode geometry on fp32 embeddings: cluster centroids + centroid-closest members, query matching.
hipError_t launch_episode_medoids(const float* emb, const int32_t* assign, int K, int E, int D,
                                  float* centroids, int32_t* medoid, hipStream_t stream);
hipError_t launch_match_queries(const float* queries, const float* centroids, int nq, int E, int D, float tau,
                                int32_t* episode, float* cosine_opt, hipStream_t stream);

}  // namespace epicache

// In-place, order-preserving compaction of the K and V caches (the cache returns
// to M entries after each block, paper Sec. 2.2 and App. A.3): row j of every
// (batch item, KV head) becomes row keep[j], keep strictly ascending.
//
// Hazard of doing this in place: keep[j] >= j, so the destination rows of one
// part of the job are the source rows of another.  compact_rows therefore cuts
// the job only along axes that never alias - (batch item, head), K vs V, and
// 16-byte column slices of the head_dim row - and each workgroup walks its rows
// in ascending chunks: all loads of a chunk, a barrier, then its stores.  A later
// chunk only reads rows at or beyond its own first destination row, which no
// earlier chunk writes, so chunks need no further ordering.  select_compact cuts
// along the rows as well and orders the parts by what they report to each other.
#include "epicache_internal.h"
#include "launch_rules.h"
#include "select_util.h"

namespace epicache {
namespace {

typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;

// Every byte is touched exactly once, so loads and stores are marked non-temporal: among the cache-policy
// combinations tried (nt, sc0, sc1 on loads and stores) nt on both is the fastest, 4 % ahead of the default.
__device__ __forceinline__ u32x4 load_row16(const unsigned char* p) {
  return __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));
}
__device__ __forceinline__ void store_row16(unsigned char* p, u32x4 v) {
  __builtin_nontemporal_store(v, reinterpret_cast<u32x4*>(p));
}

// Ragged batch: this head's own count, never beyond the pitch of its index row.
__device__ __forceinline__ int rows_kept(const Plan& pl, int bh) {
  if (!pl.n_kept) return pl.n_keep;
  const int n = pl.n_kept[bh];
  return n < 0 ? 0 : (n > pl.keep_stride ? pl.keep_stride : n);
}

// kUnroll row rounds in flight per thread, 16 bytes each.
//
// Bound by HBM where there are enough (batch item, head) pairs, by the length of a workgroup's chain of chunks where
// there are few; large workgroups serve both: a chunk of 1024 threads x 8 rounds is 128 KB.  Read + written at N = 4096,
// M = 2048, d = 128 bf16: 896 heads 358 us (256 threads x 8) -> 338 us (1024 x 4) = 5.6 TB/s; 32 heads 21.2 -> 14.1 us
// (1024 x 8, four 64-byte slices instead of two of 128).
template <int kThreads, int kUnroll>
__global__ __launch_bounds__(kThreads) void compact_rows(unsigned char* __restrict__ kbuf,
                                                    unsigned char* __restrict__ vbuf,
                                                    const int32_t* __restrict__ keep, Plan pl,
                                                    int slices, int tpr) {
  // The slices of one (bh, tensor) share cache lines and are given ids that land on one XCD (ids are dealt to the 8
  // XCDs round-robin): id = xcd + 8 * (slice + slices * (problem / 8)), problem = tensor + 2 * bh, problem % 8 = xcd.
  const int within = blockIdx.x >> 3;
  const int slice = within % slices;
  const int problem = within / slices * 8 + (blockIdx.x & 7);
  const int tensor = problem & 1, bh = problem >> 1;
  if (bh >= pl.nb * pl.Hkv) return;
  const int b = batch_of(pl, bh), h = bh - b * pl.Hkv;
  const int rpr = kThreads / tpr;            // rows per round
  const int rr = threadIdx.x / tpr, col = threadIdx.x % tpr;
  const bool lane_on = rr < rpr;
  const size_t pitch = (size_t)pl.kst * pl.elem;
  unsigned char* base = (tensor ? vbuf : kbuf) + ((size_t)b * pl.ksb + (size_t)h * pl.ksh) * pl.elem +
                        ((size_t)slice * tpr + col) * 16;
  const int32_t* idx = keep + (size_t)bh * pl.keep_stride;
  const int n = rows_kept(pl, bh);
  const int chunk = kUnroll * rpr;

  int src[kUnroll];
  auto load_idx = [&](int c0) {
#pragma unroll
    for (int u = 0; u < kUnroll; u++) {
      const int j = c0 + u * rpr + rr;
      src[u] = (lane_on && j < n) ? idx[j] : -1;
    }
  };
  load_idx(0);
  for (int c0 = 0; c0 < n; c0 += chunk) {
    u32x4 data[kUnroll];
    int cur[kUnroll];
#pragma unroll
    for (int u = 0; u < kUnroll; u++) {
      cur[u] = src[u];
      // Rows already in place (a kept prefix) are neither read nor written.  An index outside [0, N) (not one
      // epicache_topk writes) is skipped like the -1 of an idle lane, so no access leaves the rows the strides
      // were validated for.
      if ((unsigned)cur[u] >= (unsigned)pl.N) cur[u] = -1;
      if (cur[u] >= 0 && cur[u] != c0 + u * rpr + rr)
        data[u] = load_row16(base + (size_t)cur[u] * pitch);
    }
    if (c0 + chunk < n) load_idx(c0 + chunk);
    __syncthreads();  // every load of this chunk has landed before any of its stores
#pragma unroll
    for (int u = 0; u < kUnroll; u++) {
      const int j = c0 + u * rpr + rr;
      if (cur[u] >= 0 && cur[u] != j) store_row16(base + (size_t)j * pitch, data[u]);
    }
  }
}

// Ranges of kept rows of one (batch item, head) and tensor, each in the registers of one workgroup (kRounds times 16 bytes per
// thread): src[u] is the row that the thread has a part of in round u, or -1 for none, and goes to first + u * rpr + rr.
// Rows of a lower range may come from where a higher one goes, so a workgroup stores once all lower ranges are in their
// workgroups' registers.  The ranges are taken in the order in which the workgroups start (claims), so each waits only for
// workgroups that are running and that wait for nothing before they report: the wait ends whatever else the GPU runs.
// The report needs no order with other memory: the loads' values are in registers when it is made.
// The claims are memory of the caller, though.  Another call that is not ordered with this one may clear or overwrite them
// while they are in use: a range that does not exist is none, and a workgroup that has looked `patience` times leaves its
// rows as they are.
// moving_lds: null, or whether the range has a row that is not in its place; if not, it has nothing to wait for.
template <int kRounds>
__device__ __forceinline__ void load_range(u32x4 (&data)[kRounds], const int (&src)[kRounds], const unsigned char* rows, size_t pitch) {
#pragma unroll
  for (int u = 0; u < kRounds; u++)
    if (src[u] >= 0) data[u] = load_row16(rows + (size_t)src[u] * pitch);
}
template <int kRounds>
__device__ __forceinline__ void store_range(u32x4 (&data)[kRounds], const int (&src)[kRounds], unsigned char* rows, size_t pitch,
                                            int to, int rpr, uint32_t* reported, int part, bool alone, int patience,
                                            uint32_t* missing_lds, const uint32_t* moving_lds) {
#pragma unroll
  for (int u = 0; u < kRounds; u++) asm volatile("" : "+v"(data[u]) : : "memory");
  __syncthreads();  // every load of this part has landed
  if (moving_lds && !*moving_lds) {
    if (threadIdx.x == 0 && !alone) __hip_atomic_fetch_or(reported, 1u << part, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return;
  }
  if (!alone) {
    if (threadIdx.x == 0) {
      __hip_atomic_fetch_or(reported, 1u << part, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      const uint32_t below = (1u << part) - 1;
      auto missing = [&] { return below & ~__hip_atomic_load(reported, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
      uint32_t left = missing();
      for (int looks = 0; left && looks < patience; looks++) {
        __builtin_amdgcn_s_sleep(1);
        left = missing();
      }
      *missing_lds = left;
    }
    __syncthreads();
    if (*missing_lds) return;
  }
#pragma unroll
  for (int u = 0; u < kRounds; u++)
    if (src[u] >= 0) store_row16(rows + (size_t)(to + u * rpr) * pitch, data[u]);
}

// The rows of a (batch item, head) and tensor in ranges instead of one workgroup's chunks (or one's for every 64-byte slice of them):
// bound by HBM for few heads too.  8 heads, 10809 of 18363 rows of 256 bytes: 49.7 us in compact_rows, 16.9 here; 896
// heads, 2048 of 4096: 323 us (5.8 TB/s), 291 (6.5).
// Rows in their places cost a range its start only: it reports without a wait, and those of a head of which no row moves leave at once (760
// ragged heads, 4138 of 4273 rows, most of them kept again: whole step 446 us with compact_rows, 533 where such ranges wait in turn, 423).
// kLeave: heads of a ragged batch with more workgroups than ranges; those leave before they take one.
template <int kThreads, int kRounds, bool kLeave>
__global__ __launch_bounds__(kThreads, 4) void compact_ranges(unsigned char* __restrict__ kbuf, unsigned char* __restrict__ vbuf,
                                                           const int32_t* __restrict__ keep, uint32_t* claims, Plan pl, int parts,
                                                           int per_part, int tpr, int patience) {
  __shared__ uint32_t claim, moving;
  const int problems = pl.nb * pl.Hkv * 2;
  const int problem = blockIdx.x % problems;  // all heads' lowest ranges first
  const int tensor = problem & 1, bh = problem >> 1;
  const int n = rows_kept(pl, bh);
  bool one = parts == 1;  // there is nothing to take
  int32_t last = -1;
  if constexpr (kLeave) {
    if ((int)(blockIdx.x / problems) * per_part >= n) return;
    one = n <= per_part;
    // a selection's indices ascend: with the last one in its place all are, and no range of the head moves or waits
    last = keep[(size_t)bh * pl.keep_stride + n - 1];  // on its way beside the claim
  }
  uint32_t* mine = claims + (size_t)bh * kClaimsPerHead + tensor * 2 * kClaimPitch;
  if (threadIdx.x == 0) {
    moving = 0;
    claim = one ? 0 : __hip_atomic_fetch_add(mine, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __syncthreads();
  if (kLeave && last == n - 1) return;
  const int part = __builtin_amdgcn_readfirstlane(claim);
  if ((uint32_t)part >= (uint32_t)parts || part * per_part >= n) return;
  const bool alone = n <= per_part;
  const int first = part * per_part, count = min(per_part, n - first);
  const int b = batch_of(pl, bh), h = bh - b * pl.Hkv;
  const int rpr = kThreads / tpr;  // rows per round
  const int rr = threadIdx.x / tpr, col = threadIdx.x % tpr;
  const size_t pitch = (size_t)pl.kst * pl.elem;
  unsigned char* rows = (tensor ? vbuf : kbuf) + ((size_t)b * pl.ksb + (size_t)h * pl.ksh) * pl.elem + (size_t)col * 16;
  const int32_t* idx = keep + (size_t)bh * pl.keep_stride + first;
  int src[kRounds];
#pragma unroll
  for (int u = 0; u < kRounds; u++) {
    const int i = u * rpr + rr;
    src[u] = rr < rpr && i < count ? idx[i] : -1;
  }
#pragma unroll
  for (int u = 0; u < kRounds; u++) {
    // a row in place is neither read nor written; an index that no selection writes is skipped
    if (src[u] == first + u * rpr + rr || (unsigned)src[u] >= (unsigned)pl.N) src[u] = -1;
    asm volatile("" : "+v"(src[u]));  // kept as a number; masks of all rounds do not fit the scalar registers
  }
  u32x4 data[kRounds];
  load_range<kRounds>(data, src, rows, pitch);
  bool moves = false;
#pragma unroll
  for (int u = 0; u < kRounds; u++) moves |= src[u] >= 0;
  if (moves) moving = 1;
  store_range<kRounds>(data, src, rows, pitch, first + rr, rpr, mine + kClaimPitch, part, alone, patience, &claim, &moving);
}

// Selection and compaction in one: the step of few heads, where a launch of its own for either is mostly its start.
//
// A (batch item, head) and tensor is cut into `parts` ranges of kept rows, each small enough for the registers of one
// workgroup (kRounds times 16 bytes per thread).  Every workgroup does its head's whole selection for itself (the scores
// come from L2, and the search is as long for one as for all), writes the kept indices of its own range into LDS, loads
// those rows, and stores them.
template <int kThreads, int VPT, int kRounds>
__global__ __launch_bounds__(kThreads, 4) void select_compact(const float* __restrict__ scores, int32_t* __restrict__ keep,
                                                           unsigned char* __restrict__ kbuf, unsigned char* __restrict__ vbuf,
                                                           uint32_t* claims, Plan pl, int n_scored, int n_select,
                                                           int n_total, int parts, int tpr, int spread, int patience) {
  constexpr int NW = kThreads / 64;
  __shared__ SelectLds<NW> sm;
  __shared__ int32_t list[kThreads * kRounds];
  __shared__ uint32_t claim;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // the parts of one (bh, tensor) on one XCD, as the slices above, or (spread) on all of them
  const int problem = spread ? blockIdx.x % (2 * pl.nb * pl.Hkv) : (blockIdx.x >> 3) / parts * 8 + (blockIdx.x & 7);
  const int tensor = problem & 1, bh = problem >> 1;
  if (bh >= pl.nb * pl.Hkv) return;
  uint32_t* mine = claims + (size_t)bh * kClaimsPerHead + tensor * 2 * kClaimPitch;
  uint32_t taken = 0;
  if (tid == 0 && parts > 1) taken = __hip_atomic_fetch_add(mine, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  uint32_t keys[VPT], least;
  const int base = wave * VPT * 64 + lane;
  load_keys(keys, least, scores + (size_t)bh * n_scored, base, n_scored);
  if (tid == 0) claim = taken;
  const Threshold t = select_threshold<VPT, NW>(keys, least, n_scored, (uint32_t)n_select, wave, lane, sm);
  const int part = __builtin_amdgcn_readfirstlane(claim);
  if ((uint32_t)part >= (uint32_t)parts) return;
  const int per_part = (n_total + parts - 1) / parts;
  const int first = part * per_part, count = max(min(per_part, n_total - first), 0);
  emit_kept<VPT, NW>(keys, base, n_scored, t, [&](uint32_t place, int index) {
    const uint32_t at = place - (uint32_t)first;
    if (at < (uint32_t)count) list[at] = index;
  }, wave, 0, lane, sm);
  // rows kept whatever they score come behind the selected ones
  for (int i = max(n_select - first, 0) + tid; i < count; i += kThreads) list[i] = n_scored + first + i - n_select;
  __syncthreads();

  const int b = batch_of(pl, bh), h = bh - b * pl.Hkv;
  const int rpr = kThreads / tpr;  // rows per round
  const int rr = tid / tpr, col = tid % tpr;
  const size_t pitch = (size_t)pl.kst * pl.elem;
  unsigned char* rows = (tensor ? vbuf : kbuf) + ((size_t)b * pl.ksb + (size_t)h * pl.ksh) * pl.elem + (size_t)col * 16;
  u32x4 data[kRounds];
  int src[kRounds];  // -1: no row, or one in place, which is neither read nor written
#pragma unroll
  for (int u = 0; u < kRounds; u++) {
    const int i = u * rpr + rr;
    src[u] = rr < rpr && i < count ? list[i] : -1;
    if (src[u] == first + i) src[u] = -1;
    asm volatile("" : "+v"(src[u]));  // kept as a number; masks of all rounds do not fit the scalar registers
  }
  load_range<kRounds>(data, src, rows, pitch);
  if (tensor == 0 && keep)
    for (int i = tid; i < count; i += kThreads) keep[(size_t)bh * pl.keep_stride + first + i] = list[i];
  store_range<kRounds>(data, src, rows, pitch, first + rr, rpr, mine + kClaimPitch, part, parts == 1, patience, &claim, nullptr);
}

__global__ void clear_all_claims(uint32_t* claims, int heads) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < heads * 4) claims[(size_t)i * kClaimPitch] = 0;
}

}  // namespace

hipError_t launch_clear_claims(uint32_t* claims, int heads, hipStream_t stream) {
  static_assert(kClaimsPerHead == 4 * kClaimPitch, "");
  hipLaunchKernelGGL(clear_all_claims, dim3((heads * 4 + 255) / 256), dim3(256), 0, stream, claims, heads);
  return hipGetLastError();
}

hipError_t launch_select_compact(const Plan& scored, const Plan& cache, const float* scores, int32_t* keep_opt, int appended,
                                 void* k, void* v, hipStream_t stream, bool* done, int patience) {
  *done = false;
  if (!scored.claims || scored.N <= scored.M) return hipSuccess;
  const int n_total = scored.n_keep + appended, tpr = cache.d * cache.elem / 16;
  const int64_t problems = (int64_t)cache.nb * cache.Hkv * 2;
  const int parts = select_compact_parts(problems, scored.N, n_total, tpr * 16);
  if (parts == 0) return hipSuccess;
  const int threads = select_compact_threads(scored.N), per_round = threads / tpr;  // rows
  const bool spread = spreads_ranges(problems, parts);
  const dim3 grid((unsigned)((spread ? problems : (problems + 7) / 8 * 8) * parts));
  auto launch = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, grid, dim3(threads), 0, stream, scores, keep_opt, static_cast<unsigned char*>(k),
                       static_cast<unsigned char*>(v), scored.claims, cache, scored.N, scored.n_keep, n_total, parts, tpr,
                       (int)spread, patience);
  };
  // Eight rounds leave the registers for two workgroups per CU; sixteen are for those that would otherwise be two (24 heads, 3000
  // of 4336 rows: 27.4 us in ten parts of eight rounds, 21.3 in five of sixteen).
  const bool few = (n_total + parts - 1) / parts <= 8 * per_round;  // rows of a part
  if (scored.N <= 2048) few ? launch(select_compact<512, 4, 8>) : launch(select_compact<512, 4, 16>);
  else if (scored.N <= 4096) few ? launch(select_compact<1024, 4, 8>) : launch(select_compact<1024, 4, 16>);
  else if (scored.N <= 8192) few ? launch(select_compact<1024, 8, 8>) : launch(select_compact<1024, 8, 16>);
  else few ? launch(select_compact<1024, 16, 8>) : launch(select_compact<1024, 16, 16>);
  *done = true;
  return hipGetLastError();
}

hipError_t launch_compact(const Plan& pl, const int32_t* keep, void* k, void* v, bool beside_scoring,
                          hipStream_t stream) {
  if (!pl.n_kept && pl.N <= pl.M) return hipSuccess;  // nothing is evicted, rows stay where they are
  const int row_chunks = pl.d * pl.elem / 16;  // 16-byte chunks per row (head_dim % 8 == 0)
  const int64_t problems = (int64_t)pl.nb * pl.Hkv * 2;
  CompactRanges ranges = {0, 0};
  if (pl.claims && !beside_scoring)
    ranges = compact_ranges_of(problems, pl.n_keep, pl.n_kept ? pl.keep_stride : pl.n_keep, row_chunks * 16, pl.n_kept != nullptr);
  if (ranges.parts) {
    const bool few = ranges.rows <= 8 * (1024 / row_chunks), leave = pl.n_kept && problems * ranges.parts > 2 * kComputeUnits;
    const auto kernel = !few ? compact_ranges<1024, 16, false> : leave ? compact_ranges<1024, 8, true> : compact_ranges<1024, 8, false>;
    hipLaunchKernelGGL(kernel, dim3((unsigned)(problems * ranges.parts)), dim3(1024), 0,
                       stream, static_cast<unsigned char*>(k), static_cast<unsigned char*>(v), keep, pl.claims, pl, ranges.parts,
                       ranges.rows, row_chunks, kClaimPatience);
    return hipGetLastError();
  }
  const int slices = row_slices(problems, row_chunks * 16);
  const int tpr = row_chunks / slices;
  const dim3 grid((unsigned)((problems + 7) / 8 * 8 * slices));
  auto launch = [&](auto kernel, int threads) {
    hipLaunchKernelGGL(kernel, grid, dim3(threads), 0, stream, static_cast<unsigned char*>(k),
                       static_cast<unsigned char*>(v), keep, pl, slices, tpr);
  };
  if (beside_scoring) launch(compact_rows<256, 8>, 256);  // one wave of 64 registers fits on a SIMD next to two of scoring
  else if ((int64_t)pl.keep_stride * tpr <= 4096) launch(compact_rows<512, 4>, 512);  // few rows: two or three chunks
  else if (problems * slices <= 256) launch(compact_rows<1024, 8>, 1024);  // one workgroup per CU: as much in flight as fits
  else launch(compact_rows<1024, 4>, 1024);
  return hipGetLastError();
}

}  // namespace epicache

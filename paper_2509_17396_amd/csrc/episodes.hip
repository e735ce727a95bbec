// Episode geometry on segment embeddings (paper Sec. 3.1): centroid and centroid-closest member of
// every cluster (Stage 1, Eq. 3) and query-to-episode matching (Stage 3a; Stage 3b's rule that a
// query below the similarity threshold opens a new episode).  Small, latency-bound kernels: the
// inputs are a few thousand embedding vectors at most.
//
// All sums have a fixed order, so results repeat exactly.
#include <type_traits>

#include "epicache_internal.h"
#include "launch_rules.h"

namespace epicache {
namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / 64;
static_assert(kWaves == kMatchWaves, "the rule counts their rounds");

// Sum over the wave, in every lane: lane permutations inside the 16-lane rows, then the four rows' totals.
__device__ __forceinline__ float wave_sum(float x) {
  auto perm = [](float v, auto ctrl) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), decltype(ctrl)::value, 0xf, 0xf, false));
  };
  x += perm(x, std::integral_constant<int, 0xB1>{});   // quad_perm [1,0,3,2]
  x += perm(x, std::integral_constant<int, 0x4E>{});   // quad_perm [2,3,0,1]
  x += perm(x, std::integral_constant<int, 0x141>{});  // row_half_mirror
  x += perm(x, std::integral_constant<int, 0x140>{});  // row_mirror
  auto row = [&](int lane) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), lane)); };
  return (row(0) + row(16)) + (row(32) + row(48));
}

// Sum of the lanes up to this one, inside the 16-lane rows and then over the rows before.  Serial work between two barriers of
// every member list: by LDS shuffles centroids and medoids of 10 clusters of 1873 segments, 1024 dims, took 13.8 us, so 13.3.
__device__ __forceinline__ int wave_prefix(int x) {
  x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);  // row_shr:1, 0 where it leaves the row
  x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);  // row_shr:2
  x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);  // row_shr:4
  x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);  // row_shr:8
  x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);  // row_bcast:15, to rows 1 and 3
  x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);  // row_bcast:31, to rows 2 and 3
  return x;
}

// (cosine, index) candidates: larger cosine wins, equal cosines go to the lower index.
__device__ __forceinline__ bool better(float c, int i, float best_c, int best_i) {
  return c > best_c || (c == best_c && i < best_i);
}

__device__ __forceinline__ float cosine_from(float dot, float sq_u, float sq_v) {
  const float den = sqrtf(sq_u) * sqrtf(sq_v);
  return den > 0.f ? dot / den : 0.f;
}

constexpr int kNoIndex = 0x7fffffff;
constexpr int kMaxDim = 8192;  // the centroid of a cluster is kept in LDS while its members are compared

// Four consecutive floats from element d of a row of `dim`, zeros beyond it; vectors only where rows allow them.
template <bool VEC>
__device__ __forceinline__ float4 load4(const float* row, int d, int dim) {
  if (VEC) return d < dim ? *reinterpret_cast<const float4*>(row + d) : make_float4(0.f, 0.f, 0.f, 0.f);
  // unconditional loads of clamped addresses, so that none waits for another
  const float x = row[min(d, dim - 1)], y = row[min(d + 1, dim - 1)], z = row[min(d + 2, dim - 1)], w = row[min(d + 3, dim - 1)];
  return make_float4(d < dim ? x : 0.f, d + 1 < dim ? y : 0.f, d + 2 < dim ? z : 0.f, d + 3 < dim ? w : 0.f);
}

// The members of cluster e among segments [k0, k0 + kListed), ascending, into LDS; every thread of a workgroup of
// THREADS calls it, and the list is complete behind its last barrier.
constexpr int kListed = 4096;
template <int THREADS>
__device__ __forceinline__ int list_members(const int32_t* __restrict__ assign, int K, int e, int k0, int* members,
                                            int* wave_count) {
  constexpr int kRounds = kListed / THREADS;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  // wave w holds the 64-segment groups w, w + waves, ..: counts go into the list order group by group
  uint64_t mask[kRounds];
#pragma unroll
  for (int r = 0; r < kRounds; r++) {
    const int k = k0 + r * THREADS + tid;
    mask[r] = __ballot(assign[min(k, K - 1)] == e && k < K);
  }
#pragma unroll
  for (int r = 0; r < kRounds; r++)
    if (lane == 0) wave_count[r * (THREADS / 64) + wave] = __popcll(mask[r]);
  __syncthreads();
  // exclusive prefix over the kListed / 64 = 64 groups: one wave, one group per lane
  if (wave == 0) {
    const int own = wave_count[lane];
    const int incl = wave_prefix(own);
    wave_count[lane] = incl - own;
    if (lane == 63) wave_count[64] = incl;
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kRounds; r++) {
    const int below = __builtin_amdgcn_mbcnt_hi((uint32_t)(mask[r] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask[r], 0));
    if (mask[r] >> lane & 1) members[wave_count[r * (THREADS / 64) + wave] + below] = k0 + r * THREADS + tid;
  }
  __syncthreads();
  return wave_count[64];
}

// Centroids: workgroup (e, j) owns dims [64 j, 64 j + 64) of cluster e.  It lists the cluster's members and its 64 groups
// of 16 threads (4 dims each) sum every 64th of them, four rows in flight; the groups' sums meet in a tree of fixed order, so
// results repeat exactly: two steps from LDS behind one barrier, four by lane permutations.  Latency-bound: 1873 segments of
// 1024 dims in 10 clusters 127 us as a sweep of all rows by one workgroup per 256 dims, 4.9 with a barrier for each step of
// the tree, 4.2 now.
constexpr int kCentroidThreads = 1024;
constexpr int kCentroidDims = 64;
template <bool VEC>
__global__ __launch_bounds__(kCentroidThreads) void episode_centroids(const float* __restrict__ emb,
                                                                     const int32_t* __restrict__ assign, int K, int D,
                                                                     float* __restrict__ centroids,
                                                                     int32_t* __restrict__ medoid) {
  __shared__ int members[kListed], wave_count[kListed / 64 + 1];
  __shared__ float sums[kCentroidThreads / 16][kCentroidDims + 4];
  const int e = blockIdx.x, tid = threadIdx.x;
  const int group = tid / 16, d = blockIdx.y * kCentroidDims + tid % 16 * 4;
  float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
  int count = 0;
  for (int k0 = 0; k0 < K; k0 += kListed) {
    const int n = list_members<kCentroidThreads>(assign, K, e, k0, members, wave_count);
    for (int i = group; i < n; i += 256) {
      float4 x[4];
#pragma unroll
      for (int u = 0; u < 4; u++) x[u] = load4<VEC>(emb + (size_t)members[min(i + u * 64, n - 1)] * D, d, D);
#pragma unroll
      for (int u = 0; u < 4; u++)
        if (i + u * 64 < n) acc.x += x[u].x, acc.y += x[u].y, acc.z += x[u].z, acc.w += x[u].w;
    }
    count += n;
    __syncthreads();  // the list is rewritten by the next round
  }
  *reinterpret_cast<float4*>(&sums[group][tid % 16 * 4]) = acc;
  __syncthreads();
  // Groups 32 apart first, then 16, .. and 1: the first two steps by a lane each, the others over the 16 lanes of a dim.
  static_assert(kCentroidThreads == 1024 && kCentroidDims == 64, "a lane per dim and four groups");
  const int dim = tid / 16, g = tid % 16;
  float total = (sums[g][dim] + sums[g + 32][dim]) + (sums[g + 16][dim] + sums[g + 48][dim]);
  auto around = [](float v, auto ctrl) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), decltype(ctrl)::value, 0xf, 0xf, false));
  };
  total += around(total, std::integral_constant<int, 0x128>{});  // row_ror:8
  total += around(total, std::integral_constant<int, 0x124>{});  // row_ror:4
  total += around(total, std::integral_constant<int, 0x122>{});  // row_ror:2
  total += around(total, std::integral_constant<int, 0x121>{});  // row_ror:1
  const int c = blockIdx.y * kCentroidDims + dim;
  if (g == 0 && c < D) centroids[(size_t)e * D + c] = count ? total / (float)count : 0.f;
  if (blockIdx.y == 0 && tid == 0) medoid[e] = -1;  // no member yet: the kernel below finds the closest one
}

// Dot products of ROWS rows with the vector `cent` in LDS (zeros behind D) and their squared norms, one wave.
template <bool VEC, int ROWS>
__device__ __forceinline__ void rows_dot_cent(const float* const (&row)[ROWS], const float* cent, int D, int lane,
                                              float (&dot)[ROWS], float (&sq)[ROWS]) {
#pragma unroll
  for (int u = 0; u < ROWS; u++) dot[u] = sq[u] = 0.f;
#pragma unroll 4
  for (int d = lane * 4; d < D; d += 256) {
    const float4 c = *reinterpret_cast<const float4*>(cent + d);
    float4 x[ROWS];
#pragma unroll
    for (int u = 0; u < ROWS; u++) x[u] = load4<VEC>(row[u], d, D);
#pragma unroll
    for (int u = 0; u < ROWS; u++) {
      dot[u] = fmaf(x[u].x, c.x, fmaf(x[u].y, c.y, fmaf(x[u].z, c.z, fmaf(x[u].w, c.w, dot[u]))));
      sq[u] = fmaf(x[u].x, x[u].x, fmaf(x[u].y, x[u].y, fmaf(x[u].z, x[u].z, fmaf(x[u].w, x[u].w, sq[u]))));
    }
  }
#pragma unroll
  for (int u = 0; u < ROWS; u++) dot[u] = wave_sum(dot[u]), sq[u] = wave_sum(sq[u]);
}

// Centroid-closest member of cluster e by gridDim.y workgroups: the centroid goes to LDS, the listed members are dealt
// to all their waves, ROWS at a time.  There is no scratch to meet in, so the workgroups meet in medoid[e] itself
// (-1 from the kernel above): a workgroup whose best member beats the one it finds there, whose cosine it takes again
// by the same arithmetic, swaps its own in.  Every swap improves the entry, so this ends, and what remains is the best
// of all in whatever order they come.  Bound by its chain of round trips, most of all those of the meeting: few large
// workgroups.  1873 segments of 1024 dims in 10 clusters: one workgroup per cluster 17 us (what one CU can read), 15 of four
// waves 12.3, 3 of sixteen 8.8; both calls of 24 clusters of 4000 segments, 384 dims, 22.5 -> 17.9.
// The centroid's squared norm is one sum per lane over every 64th dim: its order decides between members whose cosines agree to the
// last bit, so it stays.  Each wave takes it once, eight reads of LDS ahead of the sums.  This launch and the one before, a read
// per sum / eight ahead: 13.1 / 12.6 us, 15 clusters of 900 segments, 1536 dims 14.9 / 14.2, 8 of 2000, 4096 dims (workgroups of
// four waves) 25.9 / 22.7, 300 of 3000, 1024 dims 29.6 / 29.3.
template <bool VEC, int THREADS, int ROWS>
__global__ __launch_bounds__(THREADS) void episode_medoids(const float* __restrict__ emb,
                                                           const int32_t* __restrict__ assign, int K, int D,
                                                           const float* __restrict__ centroids,
                                                           int32_t* __restrict__ medoid) {
  constexpr int kRows = ROWS, kMedoidThreads = THREADS, kMedoidWaves = THREADS / 64;
  extern __shared__ float cent[];  // [D rounded up to 256], zeros behind D
  __shared__ int members[kListed], wave_count[kListed / 64 + 1];
  __shared__ float sc[kMedoidWaves];
  __shared__ int si[kMedoidWaves];
  const int e = blockIdx.x, tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  for (int d = tid; d < (D + 255) / 256 * 256; d += kMedoidThreads) cent[d] = d < D ? centroids[(size_t)e * D + d] : 0.f;
  const int worker = blockIdx.y * kMedoidWaves + wave, workers = gridDim.y * kMedoidWaves;
  float csq = 0.f, best_c = -INFINITY;
  int best_i = kNoIndex;
  for (int k0 = 0; k0 < K; k0 += kListed) {
    const int n = list_members<kMedoidThreads>(assign, K, e, k0, members, wave_count);  // its barriers cover cent[]
    if (k0 == 0) {
#pragma unroll 2
      for (int d = lane; d < D; d += 256) {
        float c[4];
#pragma unroll
        for (int j = 0; j < 4; j++) c[j] = cent[d + j * 64];
#pragma unroll
        for (int j = 0; j < 4; j++) csq = fmaf(c[j], c[j], csq);
      }
      csq = wave_sum(csq);
    }
    for (int i = worker; i < n; i += workers * kRows) {
      float dot[kRows], sq[kRows];
      const float* row[kRows];
#pragma unroll
      for (int u = 0; u < kRows; u++) row[u] = emb + (size_t)members[min(i + u * workers, n - 1)] * D;
      rows_dot_cent<VEC, kRows>(row, cent, D, lane, dot, sq);
#pragma unroll
      for (int u = 0; u < kRows; u++) {
        const int at = i + u * workers;
        if (at >= n) continue;
        const float c = cosine_from(dot[u], sq[u], csq);
        const int k = members[at];
        if (better(c, k, best_c, best_i)) best_c = c, best_i = k;
      }
    }
    __syncthreads();  // the list is rewritten by the next round
  }
  if (lane == 0) sc[wave] = best_c, si[wave] = best_i;
  __syncthreads();
  if (wave != 0) return;
  best_c = sc[lane % kMedoidWaves], best_i = si[lane % kMedoidWaves];
#pragma unroll
  for (int off = kMedoidWaves / 2; off >= 1; off /= 2) {
    const float c = __shfl_xor(best_c, off);
    const int i = __shfl_xor(best_i, off);
    if (better(c, i, best_c, best_i)) best_c = c, best_i = i;
  }
  if (best_i == kNoIndex) return;  // no member here; an empty cluster keeps its -1
  int held = -1;  // as the first one finds it
  while (true) {
    if (held >= 0) {
      float dot[1], sq[1];
      const float* row[1] = {emb + (size_t)held * D};
      rows_dot_cent<VEC, 1>(row, cent, D, lane, dot, sq);
      if (!better(best_c, best_i, cosine_from(dot[0], sq[0], csq), held)) break;
    }
    int seen = held;
    if (lane == 0) seen = atomicCAS(medoid + e, held, best_i);
    seen = __builtin_amdgcn_readfirstlane(seen);
    if (seen == held) break;
    held = seen;
  }
}

// One workgroup per query; the centroids are dealt to its waves, ROWS of a wave's at a time (match_rows).
template <bool VEC, int ROWS>
__global__ __launch_bounds__(kThreads) void match_queries(const float* __restrict__ queries,
                                                          const float* __restrict__ centroids, int E, int D,
                                                          float tau, int32_t* __restrict__ episode,
                                                          float* __restrict__ cosine_opt) {
  constexpr int kRows = ROWS;
  __shared__ float sc[kWaves];
  __shared__ int si[kWaves];
  const int qi = blockIdx.x, tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const float* q = queries + (size_t)qi * D;
  float best_c = -INFINITY;
  int best_i = kNoIndex;
  for (int e = wave; e < E; e += kWaves * kRows) {
    float dot[kRows], sq[kRows], qsq = 0.f;
    const float* row[kRows];
#pragma unroll
    for (int u = 0; u < kRows; u++) dot[u] = sq[u] = 0.f, row[u] = centroids + (size_t)min(e + u * kWaves, E - 1) * D;
#pragma unroll 4
    for (int d = lane * 4; d < D; d += 256) {
      const float4 y = load4<VEC>(q, d, D);
      float4 x[kRows];
#pragma unroll
      for (int u = 0; u < kRows; u++) x[u] = load4<VEC>(row[u], d, D);
      qsq = fmaf(y.x, y.x, fmaf(y.y, y.y, fmaf(y.z, y.z, fmaf(y.w, y.w, qsq))));
#pragma unroll
      for (int u = 0; u < kRows; u++) {
        dot[u] = fmaf(x[u].x, y.x, fmaf(x[u].y, y.y, fmaf(x[u].z, y.z, fmaf(x[u].w, y.w, dot[u]))));
        sq[u] = fmaf(x[u].x, x[u].x, fmaf(x[u].y, x[u].y, fmaf(x[u].z, x[u].z, fmaf(x[u].w, x[u].w, sq[u]))));
      }
    }
    qsq = wave_sum(qsq);
#pragma unroll
    for (int u = 0; u < kRows; u++) dot[u] = wave_sum(dot[u]), sq[u] = wave_sum(sq[u]);
#pragma unroll
    for (int u = 0; u < kRows; u++) {
      const int at = e + u * kWaves;
      const float c = cosine_from(dot[u], qsq, sq[u]);
      if (at < E && better(c, at, best_c, best_i)) best_c = c, best_i = at;
    }
  }
  if (lane == 0) sc[wave] = best_c, si[wave] = best_i;
  __syncthreads();
  if (tid == 0) {
    float c = sc[0];
    int i = si[0];
    for (int w = 1; w < kWaves; w++)
      if (better(sc[w], si[w], c, i)) c = sc[w], i = si[w];
    episode[qi] = c >= tau ? i : -1;
    if (cosine_opt) cosine_opt[qi] = c;
  }
}

}  // namespace

// Rows that all start on 16 bytes.
static bool vector_rows(const float* a, const float* b, int D) {
  return D % 4 == 0 && ((reinterpret_cast<uintptr_t>(a) | reinterpret_cast<uintptr_t>(b)) & 15) == 0;
}

hipError_t launch_episode_medoids(const float* emb, const int32_t* assign, int K, int E, int D,
                                  float* centroids, int32_t* medoid, hipStream_t stream) {
  if (D > kMaxDim) return hipErrorInvalidValue;
  const dim3 grid(E, (D + kCentroidDims - 1) / kCentroidDims);
  const size_t smem = (size_t)((D + 255) / 256 * 256) * sizeof(float);
  const MedoidShape shape = medoid_shape(K, E, D);
  auto launch = [&](auto centroid_kernel, auto medoid_kernel) {
    hipLaunchKernelGGL(centroid_kernel, grid, dim3(kCentroidThreads), 0, stream, emb, assign, K, D, centroids,
                       medoid);
    hipLaunchKernelGGL(medoid_kernel, dim3(E, shape.per_cluster), dim3(shape.threads), smem, stream, emb, assign, K, D, centroids,
                       medoid);
  };
  const bool vec = vector_rows(emb, emb, D), large = shape.threads == 1024;
  if (vec) launch(episode_centroids<true>, large ? episode_medoids<true, 1024, 4> : episode_medoids<true, 256, 3>);
  else launch(episode_centroids<false>, large ? episode_medoids<false, 1024, 4> : episode_medoids<false, 256, 3>);
  return hipGetLastError();
}

hipError_t launch_match_queries(const float* queries, const float* centroids, int nq, int E, int D, float tau,
                                int32_t* episode, float* cosine_opt, hipStream_t stream) {
  const bool vec = vector_rows(queries, centroids, D), three = match_rows(nq, E) == 3;
  const auto kernel = vec ? (three ? match_queries<true, 3> : match_queries<true, 2>)
                          : (three ? match_queries<false, 3> : match_queries<false, 2>);
  hipLaunchKernelGGL(kernel, dim3(nq), dim3(kThreads), 0, stream, queries, centroids, E, D, tau, episode, cosine_opt);
  return hipGetLastError();
}

}  // namespace epicache

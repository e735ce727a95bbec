// KeyDiff scoring (paper App. A.2, "KeyDiff"): an attention-free scorer for the same select /
// compact back end.  Per (batch item, KV head): anchor = mean of the N context keys, score of row i
// = -cos(k_i, anchor).  A zero key or a zero anchor has cosine 0.
//
// One pass over K where a row is read by 8 or 16 lanes (bf16 d = 64/128, fp32 d = 32/64) and a head fits 64 workgroups:
// keydiff_fused.  Otherwise two streaming passes, both HBM-bound:
//   keydiff_partial: column sums of 512-row chunks, one workgroup per chunk, written to the workspace
//                    (no atomics: the chunk sums are added in a fixed order, so results repeat exactly);
//   keydiff_scores:  every workgroup rebuilds the anchor from the chunk sums (a few KB from L2), then
//                    computes dot(k_i, anchor) and |k_i|^2 for its rows.
// A row is read by d*elem/16 threads with one 16-byte load each.  When those are 8 or 16 lanes the per-row sums are
// reduced with in-register lane permutations and the scores of a chunk leave through LDS as one contiguous run; other
// head dims meet in LDS.
#include <hip/hip_bf16.h>

#include <type_traits>

#include "epicache_internal.h"

namespace epicache {
namespace {

constexpr int kThreads = 256;
constexpr int kChunkRows = 512;  // rows per workgroup in both passes
constexpr int kUnroll = 8;       // row rounds in flight per thread in the scoring pass

template <typename T>
struct Vec;
template <>
struct Vec<float> {
  static constexpr int kLen = 4;
  __device__ static void unpack(const uint4& v, float (&x)[4]) {
    x[0] = __uint_as_float(v.x), x[1] = __uint_as_float(v.y);
    x[2] = __uint_as_float(v.z), x[3] = __uint_as_float(v.w);
  }
  __device__ static void load(const void* p, float (&x)[4]) { unpack(*reinterpret_cast<const uint4*>(p), x); }
};
template <>
struct Vec<__hip_bfloat16> {
  static constexpr int kLen = 8;
  __device__ static void unpack(const uint4& v, float (&x)[8]) {
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int i = 0; i < 4; i++) {
      x[2 * i] = __uint_as_float(w[i] << 16);          // bf16 -> fp32: the bits, shifted up
      x[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
    }
  }
  __device__ static void load(const void* p, float (&x)[8]) { unpack(*reinterpret_cast<const uint4*>(p), x); }
};

template <typename T>
__global__ __launch_bounds__(kThreads) void keydiff_partial(const T* __restrict__ k,
                                                            float* __restrict__ partial, Plan pl, int chunks) {
  constexpr int VL = Vec<T>::kLen;
  __shared__ float sm[kThreads * VL];
  const int bh = blockIdx.y, b = bh / pl.Hkv, h = bh % pl.Hkv;
  const int N = ctx_rows(pl, bh);
  const int tpr = pl.d / VL, rpr = kThreads / tpr;
  const int rr = threadIdx.x / tpr, col = threadIdx.x % tpr;
  const int row0 = blockIdx.x * kChunkRows;
  const int row_end = min(N, row0 + kChunkRows);
  const unsigned char* base = reinterpret_cast<const unsigned char*>(k + b * pl.ksb + (int64_t)h * pl.ksh) +
                              (size_t)col * 16;
  const size_t pitch = (size_t)pl.kst * sizeof(T);
  float acc[VL];
#pragma unroll
  for (int e = 0; e < VL; e++) acc[e] = 0.f;
  if (rr < rpr) {
    int row = row0 + rr;
    for (; row + 7 * rpr < row_end; row += 8 * rpr) {  // eight loads in flight per thread
      float x[8][VL];
#pragma unroll
      for (int u = 0; u < 8; u++) Vec<T>::load(base + (size_t)(row + u * rpr) * pitch, x[u]);
#pragma unroll
      for (int u = 0; u < 8; u++)
#pragma unroll
        for (int e = 0; e < VL; e++) acc[e] += x[u][e];
    }
    for (; row < row_end; row += rpr) {
      float x[VL];
      Vec<T>::load(base + (size_t)row * pitch, x);
#pragma unroll
      for (int e = 0; e < VL; e++) acc[e] += x[e];
    }
#pragma unroll
    for (int e = 0; e < VL; e++) sm[rr * pl.d + col * VL + e] = acc[e];
  }
  __syncthreads();
  for (int c = threadIdx.x; c < pl.d; c += kThreads) {
    float s = 0.f;
    for (int g = 0; g < rpr; g++) s += sm[g * pl.d + c];
    partial[((size_t)bh * chunks + blockIdx.x) * pl.d + c] = s;
  }
}

// Sum over the 8 or 16 consecutive lanes that share a row, with data-parallel-primitive lane
// permutations inside a 16-lane row (no LDS traffic): lane pairs (i, i^1), (i, i^2), then i <-> 7-i
// within each half row and i <-> 15-i within the row.  Every lane of the group ends with the total.
template <int LANES>
__device__ __forceinline__ float group_sum(float x) {
  auto perm = [](float v, auto ctrl) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), decltype(ctrl)::value, 0xf, 0xf, false));
  };
  x += perm(x, std::integral_constant<int, 0xB1>{});   // quad_perm [1,0,3,2]
  x += perm(x, std::integral_constant<int, 0x4E>{});   // quad_perm [2,3,0,1]
  x += perm(x, std::integral_constant<int, 0x141>{});  // row_half_mirror
  if (LANES == 16) x += perm(x, std::integral_constant<int, 0x140>{});  // row_mirror
  return x;
}

// IN_WAVE: d*elem/16 is 8 or 16, so the lanes of a row sit inside one 16-lane row of a wave.
template <typename T, bool IN_WAVE>
__global__ __launch_bounds__(kThreads) void keydiff_scores(const T* __restrict__ k,
                                                           const float* __restrict__ partial,
                                                           float* __restrict__ scores, Plan pl, int chunks) {
  constexpr int VL = Vec<T>::kLen;
  __shared__ float anchor[256];
  __shared__ float anchor_norm;
  __shared__ float red_dot[kUnroll][kThreads], red_sq[kUnroll][kThreads];
  __shared__ float out[kChunkRows];
  const int bh = blockIdx.y, b = bh / pl.Hkv, h = bh % pl.Hkv;
  const int N = ctx_rows(pl, bh);
  const int row0 = blockIdx.x * kChunkRows;
  if (row0 >= N) return;
  const int tid = threadIdx.x;
  const int tpr = pl.d / VL, rpr = kThreads / tpr;
  const int rr = tid / tpr, col = tid % tpr;

  const unsigned char* base = reinterpret_cast<const unsigned char*>(k + b * pl.ksb + (int64_t)h * pl.ksh) +
                              (size_t)col * 16;
  const size_t pitch = (size_t)pl.kst * sizeof(T);
  const int row_end = min(N, row0 + kChunkRows);
  const int rows_per_iter = kUnroll * rpr;

  // raw 16-byte loads; they are widened to fp32 only when used, which keeps many loads in flight
  // at 4 registers each
  auto load_rows = [&](int it0, uint4 (&x)[kUnroll]) {
#pragma unroll
    for (int u = 0; u < kUnroll; u++) {
      const int row = it0 + u * rpr + rr;
      x[u] = make_uint4(0, 0, 0, 0);
      if (rr < rpr && row < row_end) x[u] = *reinterpret_cast<const uint4*>(base + (size_t)row * pitch);
    }
  };
  uint4 xr[kUnroll];
  if constexpr (IN_WAVE) load_rows(row0, xr);  // in flight while the anchor is rebuilt

  // anchor = (sum of the chunk sums) / N, in chunk order
  for (int c = tid; c < pl.d; c += kThreads) {
    float s = 0.f;
    for (int g = 0; g < chunks; g++) s += partial[((size_t)bh * chunks + g) * pl.d + c];
    anchor[c] = s / (float)N;
  }
  __syncthreads();
  if (tid < 64) {
    float s = 0.f;
    for (int c = tid; c < pl.d; c += 64) s = fmaf(anchor[c], anchor[c], s);
    for (int off = 32; off >= 1; off >>= 1) s += __shfl_xor(s, off);
    if (tid == 0) anchor_norm = sqrtf(s);
  }
  __syncthreads();
  const float an = anchor_norm;
  float a[VL];
#pragma unroll
  for (int e = 0; e < VL; e++) a[e] = rr < rpr ? anchor[col * VL + e] : 0.f;

  if constexpr (IN_WAVE) {
    // reduce in registers, no barrier; scores are collected in LDS and written as one contiguous run
    for (int it0 = row0; it0 < row_end; it0 += rows_per_iter) {
#pragma unroll
      for (int u = 0; u < kUnroll; u++) {
        float x[VL];
        Vec<T>::unpack(xr[u], x);
        float dot = 0.f, sq = 0.f;
#pragma unroll
        for (int e = 0; e < VL; e++) {
          dot = fmaf(x[e], a[e], dot);
          sq = fmaf(x[e], x[e], sq);
        }
        if (tpr == 16) dot = group_sum<16>(dot), sq = group_sum<16>(sq);
        else dot = group_sum<8>(dot), sq = group_sum<8>(sq);
        const int row = it0 + u * rpr + rr;
        if (col == 0 && row < row_end) {
          const float den = sqrtf(sq) * an;
          out[row - row0] = den > 0.f ? -dot / den : 0.f;
        }
        // refill this slot for the next iteration as soon as it has been consumed
        const int nrow = row + rows_per_iter;
        xr[u] = make_uint4(0, 0, 0, 0);
        if (nrow < row_end) xr[u] = *reinterpret_cast<const uint4*>(base + (size_t)nrow * pitch);
      }
    }
    __syncthreads();
    for (int j = tid; j < row_end - row0; j += kThreads) scores[(size_t)bh * pl.N + row0 + j] = out[j];
  } else {
    for (int it0 = row0; it0 < row_end; it0 += rows_per_iter) {
      float x[kUnroll][VL];  // all loads of the iteration are issued before the first use
#pragma unroll
      for (int u = 0; u < kUnroll; u++) {
        const int row = it0 + u * rpr + rr;
        if (rr < rpr && row < row_end) {
          Vec<T>::load(base + (size_t)row * pitch, x[u]);
        } else {
#pragma unroll
          for (int e = 0; e < VL; e++) x[u][e] = 0.f;
        }
      }
#pragma unroll
      for (int u = 0; u < kUnroll; u++) {
        float dot = 0.f, sq = 0.f;
#pragma unroll
        for (int e = 0; e < VL; e++) {
          dot = fmaf(x[u][e], a[e], dot);
          sq = fmaf(x[u][e], x[u][e], sq);
        }
        red_dot[u][tid] = dot;
        red_sq[u][tid] = sq;
      }
      __syncthreads();
      for (int j = tid; j < rows_per_iter; j += kThreads) {  // j-th row of this iteration
        const int u = j / rpr, g = j % rpr;
        const int row = it0 + j;
        if (row < row_end) {
          float dot = 0.f, sq = 0.f;
          for (int c = 0; c < tpr; c++) {
            dot += red_dot[u][g * tpr + c];
            sq += red_sq[u][g * tpr + c];
          }
          const float den = sqrtf(sq) * an;
          scores[(size_t)bh * pl.N + row] = den > 0.f ? -dot / den : 0.f;
        }
      }
      __syncthreads();  // the exchange buffers are rewritten by the next iteration
    }
  }
}

// Both passes in one, K read once: every workgroup keeps its rows in registers while the anchor is put together from
// the column sums of all workgroups of the head.  (Between two passes a head's K, 1 MB for 4096 rows of 128 bf16 values,
// leaves every cache.)  LANES threads hold a row, ROWS rows each.  896 heads of 4096 rows, d = 128: 332 us in two passes
// (5.7 TB/s), 196 us in one (4.8 TB/s; two to four workgroups per CU cover each other's waits).
//
// A workgroup waits for the others of its head, so it must not depend on their being resident: the wait is bounded, and
// a workgroup that gives up recomputes the sums of the head from K, in the same order and so to the same bits.  Dispatch
// goes in order of the ids and a head's workgroups have neighbouring ones, so that in practice all of them run by the time
// the first has its rows.
// The sums go through device-scope relaxed atomics (the workgroups sit on different XCDs), and every one says by itself
// whether it is there: its place holds kNotYet before.  No order between different places is asked of the memory, so no
// fences are needed, which at device scope write back and invalidate the L2 (896 heads of 4096 rows: 878 us).  The count
// of arrivals is a hint that saves looking at the sums in vain; it may run ahead of them a little, and waiting for the sums to be
// acknowledged before it costs more than the looks (12 us).  A last workgroup that adds up the sums for all costs the others
// one more round trip.  A head's workgroups on one XCD: 234 us.
constexpr int kArrivedPitch = 64;  // counters of different heads on different cache lines
constexpr uint32_t kNotYet = 0xffffffffu;  // a NaN; sums that come out as it are stored as another one

// `words` places of sums, a multiple of 4, and n counters
__global__ void keydiff_clear(uint4* sums, size_t words, uint32_t* arrived, int n) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < words / 4) sums[i] = make_uint4(kNotYet, kNotYet, kNotYet, kNotYet);
  if (i < (size_t)n) arrived[i * kArrivedPitch] = 0;
}

template <typename T, int THREADS, int LANES, int ROWS>
__global__ __launch_bounds__(THREADS, 4) void keydiff_fused(const T* __restrict__ k, uint32_t* __restrict__ partial,
                                                                 uint32_t* __restrict__ arrived,
                                                                 float* __restrict__ scores, Plan pl, int chunks,
                                                                 int patience) {
  constexpr int VL = Vec<T>::kLen, D = LANES * VL, kWaves = THREADS / 64;
  constexpr int kRound = THREADS / LANES;  // rows that the workgroup takes in with one load per thread
  constexpr int kRows = kRound * ROWS;
  __shared__ float wave_sum[kWaves][D];
  __shared__ float anchor[D];
  __shared__ float anchor_norm;
  __shared__ int complete, missing;
  __shared__ float out[kRows];
  const int bh = blockIdx.y, b = batch_of(pl, bh), h = bh - b * pl.Hkv;
  const int N = ctx_rows(pl, bh);
  const int row0 = blockIdx.x * kRows;
  if (row0 >= N) return;
  const int tid = threadIdx.x, wave = tid >> 6;
  const int rr = tid / LANES, col = tid % LANES;
  const int expected = (N + kRows - 1) / kRows;  // workgroups of this head
  const unsigned char* base = reinterpret_cast<const unsigned char*>(k + b * pl.ksb + (int64_t)h * pl.ksh) + col * 16;
  const uint32_t pitch = (uint32_t)(pl.kst * sizeof(T));

  // rows behind the last re-read it and count as zero
  auto load_row = [&](int row) { return *reinterpret_cast<const uint4*>(base + (size_t)min(row, N - 1) * pitch); };
  auto masked = [&](uint4 v, int row) { return row < N ? v : make_uint4(0, 0, 0, 0); };
  // column sums over the workgroup's rows, in threads 0 .. D - 1
  auto column_sum = [&](float (&acc)[VL]) {
#pragma unroll
    for (int e = 0; e < VL; e++) {
#pragma unroll
      for (int off = LANES; off < 64; off *= 2) acc[e] += __shfl_xor(acc[e], off);
      if ((tid & 63) < LANES) wave_sum[wave][col * VL + e] = acc[e];
    }
    __syncthreads();
    float s = 0.f;
    if (tid < D) {
#pragma unroll
      for (int w = 0; w < kWaves; w++) s += wave_sum[w][tid];
    }
    __syncthreads();
    return s;
  };

  uint4 x[ROWS];
#pragma unroll
  for (int u = 0; u < ROWS; u++) x[u] = load_row(row0 + u * kRound + rr);
  if (row0 + kRows > N) {
#pragma unroll
    for (int u = 0; u < ROWS; u++) x[u] = masked(x[u], row0 + u * kRound + rr);
  }
  float acc[VL];
#pragma unroll
  for (int e = 0; e < VL; e++) acc[e] = 0.f;
#pragma unroll
  for (int u = 0; u < ROWS; u++) {
    float v[VL];
    Vec<T>::unpack(x[u], v);
#pragma unroll
    for (int e = 0; e < VL; e++) acc[e] += v[e];
  }
  // the packed rows are what stays in registers: each use widens them again
  auto repack = [&] {
#pragma unroll
    for (int u = 0; u < ROWS; u++) asm volatile("" : "+v"(x[u].x), "+v"(x[u].y), "+v"(x[u].z), "+v"(x[u].w));
  };
  uint32_t* sums = partial + (size_t)bh * chunks * D;
  const float mine = column_sum(acc);
  if (tid < D) {
    const uint32_t bits = __float_as_uint(mine);
    __hip_atomic_store(&sums[blockIdx.x * D + tid], bits == kNotYet ? 0x7fc00000u : bits, __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
  }
  __syncthreads();
  uint32_t* count = arrived + bh * kArrivedPitch;
  if (tid == 0) __hip_atomic_fetch_add(count, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);

  repack();
  float sq[ROWS];  // squared norms, while the others arrive
#pragma unroll
  for (int u = 0; u < ROWS; u++) {
    float v[VL];
    Vec<T>::unpack(x[u], v);
    sq[u] = 0.f;
#pragma unroll
    for (int e = 0; e < VL; e++) sq[u] = fmaf(v[e], v[e], sq[u]);
    sq[u] = group_sum<LANES>(sq[u]);
  }

  repack();
  if (tid == 0) {
    bool all = false;
    for (int looks = 0; !all && looks < patience; looks++) {
      if (looks) __builtin_amdgcn_s_sleep(4);
      all = __hip_atomic_load(count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= (uint32_t)expected;
    }
    complete = all;
    missing = 0;
  }
  __syncthreads();
  // The sums of the head's workgroups in kParts runs, one per D threads, then the runs in order: a head of 16 workgroups is one
  // round trip for 256 threads (two for the first 128 of them: 896 heads of 4096 rows 4 us longer, 128 of 16384 13 us).
  constexpr int kParts = THREADS / D;
  const int run = (expected + kParts - 1) / kParts;
  __shared__ float run_sum[kParts][D];
  if (complete) {
    const int c = tid % D, first = tid / D * run, last = min(first + run, expected);
    float s = 0.f;
    int looks = 0;
    for (int g0 = first; g0 < last; g0 += 8) {
      uint32_t p[8];
      bool there;
      do {
        there = true;
        int at = g0;
        asm volatile("" : "+v"(at));  // the addresses are made again each time, not kept: the registers
#pragma unroll
        for (int g = 0; g < 8; g++)
          p[g] = __hip_atomic_load(&sums[min(at + g, last - 1) * D + c], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
        for (int g = 0; g < 8; g++) there = there && p[g] != kNotYet;
      } while (!there && looks++ < patience);
      if (!there) missing = 1;
#pragma unroll
      for (int g = 0; g < 8; g++) s += g0 + g < last ? __uint_as_float(p[g]) : 0.f;
    }
    run_sum[tid / D][c] = s;
  }
  __syncthreads();
  if (!complete || missing) {  // the head's sums from K
    for (int r = 0; r < kParts; r++) {
      float s = 0.f;
      for (int g = r * run; g < min((r + 1) * run, expected); g++) {
        for (int e = 0; e < VL; e++) acc[e] = 0.f;
        for (int u = 0; u < ROWS; u++) {
          const int row = g * kRows + u * kRound + rr;
          float v[VL];
          Vec<T>::unpack(masked(load_row(row), row), v);
          for (int e = 0; e < VL; e++) acc[e] += v[e];
        }
        s += column_sum(acc);
      }
      if (tid < D) run_sum[r][tid] = s;
    }
  }
  float s = 0.f;
  if (tid < D) {
#pragma unroll
    for (int r = 0; r < kParts; r++) s += run_sum[r][tid];
  }
  if (tid < D) anchor[tid] = s / (float)N;
  __syncthreads();
  if (tid < 64) {
    float t = 0.f;
    for (int c = tid; c < D; c += 64) t = fmaf(anchor[c], anchor[c], t);
    for (int off = 32; off >= 1; off >>= 1) t += __shfl_xor(t, off);
    if (tid == 0) anchor_norm = sqrtf(t);
  }
  float a[VL];
#pragma unroll
  for (int e = 0; e < VL; e++) a[e] = anchor[col * VL + e];
  __syncthreads();
  const float an = anchor_norm;
#pragma unroll
  for (int u = 0; u < ROWS; u++) {
    float v[VL];
    Vec<T>::unpack(x[u], v);
    float dot = 0.f;
#pragma unroll
    for (int e = 0; e < VL; e++) dot = fmaf(v[e], a[e], dot);
    dot = group_sum<LANES>(dot);
    if (col == 0) {
      const float den = sqrtf(sq[u]) * an;
      out[u * kRound + rr] = den > 0.f ? -dot / den : 0.f;
    }
  }
  __syncthreads();
  for (int j = tid; j < min(kRows, N - row0); j += THREADS) scores[(size_t)bh * pl.N + row0 + j] = out[j];
}

// How a call is cut up: threads per workgroup and rows per thread of the one-pass form (0: the two passes), workgroups
// per head.  Small workgroups overlap better (896 heads of 4096 rows: 512 threads take 5 % longer), but every one reads
// the sums of all of its head, past the caches: 1024 heads of 16384 rows 1160 us with 512 threads, with 256 1.4 times that.  Few
// rows per thread where that is what it takes to give every CU work (20 heads of 845 rows: 17.6 us in two passes, 9.8).
struct KeydiffShape {
  int threads, rows, chunks;
};
KeydiffShape keydiff_shape(const Plan& pl) {
  const int vl = pl.dtype == EPICACHE_DTYPE_F32 ? Vec<float>::kLen : Vec<__hip_bfloat16>::kLen, lanes = pl.d / vl;
  auto cut = [&](int threads, int rows) {
    const int per = threads / lanes * rows;
    return KeydiffShape{threads, rows, (pl.N + per - 1) / per};
  };
  if (lanes == 8 || lanes == 16) {
    KeydiffShape s = cut(256, 4);
    if (s.chunks <= 16 && (int64_t)s.chunks / 4 * pl.nb * pl.Hkv < 512) return s;
    s = cut(256, 16);
    if (s.chunks <= 16) return s;
    s = cut(512, 16);
    if (s.chunks <= 64) return s;
  }
  return {0, 0, (pl.N + kChunkRows - 1) / kChunkRows};
}

template <typename T>
hipError_t launch_t(const Plan& pl, const T* k, float* scores, float* partial, int patience, hipStream_t stream) {
  const KeydiffShape shape = keydiff_shape(pl);
  const int nbh = pl.nb * pl.Hkv, tpr = pl.d / Vec<T>::kLen;
  const dim3 grid(shape.chunks, nbh);
  if (shape.threads) {
    const size_t words = (size_t)nbh * shape.chunks * pl.d, threads = words / 4 > (size_t)nbh ? words / 4 : nbh;
    uint32_t* sums = reinterpret_cast<uint32_t*>(partial);
    uint32_t* arrived = sums + words;
    hipLaunchKernelGGL(keydiff_clear, dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, stream,
                       reinterpret_cast<uint4*>(sums), words, arrived, nbh);
    auto launch = [&](auto lanes) {
      constexpr int L = decltype(lanes)::value;
      auto kernel = shape.threads == 512 ? keydiff_fused<T, 512, L, 16> :
                    shape.rows == 16 ? keydiff_fused<T, 256, L, 16> : keydiff_fused<T, 256, L, 4>;
      hipLaunchKernelGGL(kernel, grid, dim3(shape.threads), 0, stream, k, sums, arrived, scores, pl, shape.chunks,
                         patience);
    };
    if (tpr == 16) launch(std::integral_constant<int, 16>{});
    else launch(std::integral_constant<int, 8>{});
    return hipGetLastError();
  }
  hipLaunchKernelGGL(keydiff_partial<T>, grid, dim3(kThreads), 0, stream, k, partial, pl, shape.chunks);
  if (tpr == 16 || tpr == 8)
    hipLaunchKernelGGL((keydiff_scores<T, true>), grid, dim3(kThreads), 0, stream, k, partial, scores, pl, shape.chunks);
  else
    hipLaunchKernelGGL((keydiff_scores<T, false>), grid, dim3(kThreads), 0, stream, k, partial, scores, pl, shape.chunks);
  return hipGetLastError();
}

}  // namespace

size_t keydiff_workspace_bytes(const Plan& pl) {
  const size_t nbh = (size_t)pl.nb * pl.Hkv;
  return nbh * keydiff_shape(pl).chunks * pl.d * sizeof(float) + nbh * kArrivedPitch * sizeof(uint32_t);
}

hipError_t launch_score_keydiff(const Plan& pl, const void* k, float* scores, void* workspace, hipStream_t stream,
                                int patience) {
  float* partial = static_cast<float*>(workspace);
  if (pl.dtype == EPICACHE_DTYPE_F32)
    return launch_t<float>(pl, static_cast<const float*>(k), scores, partial, patience, stream);
  return launch_t<__hip_bfloat16>(pl, static_cast<const __hip_bfloat16*>(k), scores, partial, patience, stream);
}

}  // namespace epicache

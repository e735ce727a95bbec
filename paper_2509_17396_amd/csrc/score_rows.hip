// Scoring with one product Q K^T, for contexts of up to 2048 rows (Eq. 1).
//
// score_mfma.hip forms every logit twice, as a row's normaliser needs all keys and its logits do not fit on chip.  With up to
// 2048 keys they do, 32 query rows at a time: 8 waves x 8 tiles of 32 x 32 weights are half of a CU's registers.  One
// workgroup takes 32 rows through all keys, sums the rows, and reduces the weights, which are still there, over the rows.
// Workgroups of one head leave their parts of its scores, which the selection adds up as it loads them: one launch less.
//
// With few heads the time is that of one workgroup's way through its keys: 64 KB per round of tiles, of which two are on their way
// (LDS holds no more, registers hold the weights), 1.3 us each behind 5 us of start and end; more workgroups for the keys of 32 rows
// would have to wait for each other's sums (1.9 us a time).  With many it is the rate at which K comes to LDS, once per 32 rows,
// and there it ends against two passes, which bring it once per 128 or 256 rows, twice (row_splits in launch_rules.h).
// Steps, us before and after: fp32, head_dim 64, 2 heads, 384 keys, 128 rows 18.3 and 16.9; bf16, head_dim 96, 64 heads, 2024 keys,
// 64 rows 31.6 and 27.5; head_dim 128, 896 heads, 2048 keys, 32 rows 275 and 188, 64 rows 278 and 218.
// Errors against float64 are no larger than those of two passes (mean of small logits 3e-8, largest 1.4e-7; 4e-8 and 1.6e-7).
#include <type_traits>

#include "epicache_internal.h"
#include "launch_rules.h"
#include "mfma_tiles.h"

namespace epicache {
namespace {

constexpr int kWaves = 8;
constexpr int kFewestTiles = 2, kMostTiles = 8;  // of 32 keys, per wave
// A weight is exp2 of its logit as it is.  Rows whose sum leaves this range, so that weights of 2^-100 of it may have been lost,
// are done again relative to their largest logit.
constexpr float kMostTotal = 0x1p100f, kLeastTotal = 0x1p-24f;

template <int N, int I = 0, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<N, I + 1>(f);
  }
}

// Values of a tile whose turn it is behind MFMA j of the next one's chain.
template <int KS> struct Slices {
  static constexpr int at(int j) { return KS == 6 ? (j < 5 ? 3 * j : j == 5 ? 14 : 16) : (16 * j) / KS; }
};
template <int LO, int HI>
__device__ __forceinline__ void slice_scale(f32x16& x, float c2) {
#pragma unroll
  for (int v = LO; v < HI; v++) {
    float y = x[v] * c2;
    pin(y);
    x[v] = y;
  }
}
template <int LO, int HI>
__device__ __forceinline__ void slice_exp(f32x16& x) {
#pragma unroll
  for (int v = LO; v < HI; v++) {
    float y = ex2(x[v]);
    pin(y);
    x[v] = y;
  }
}
template <int LO, int HI>
__device__ __forceinline__ void slice_add(const f32x16& x, float (&sum)[16]) {
#pragma unroll
  for (int v = LO; v < HI; v++) {
    sum[v] += x[v];
    pin(sum[v]);
  }
}

// The chain of one tile, a slice of the tile before behind every MFMA.
template <bool F32, int KS, int J, bool FOLD>
__device__ __forceinline__ void rows_slots(f32x16& acc, const bf16x8 (&qf)[KS], const bf16x8 (&kf)[KS], f32x16& x, float c2,
                                           float (&sum)[16]) {
  using SL = Slices<KS>;
  if (J == 0) acc = f32x16{0};
  mfma_step<F32>(acc, qf[J], kf[J]);
  fence_sched();
  if constexpr (FOLD) {
    slice_scale<SL::at(J), SL::at(J + 1)>(x, c2);
    if constexpr (J >= 1) slice_exp<SL::at(J - 1), SL::at(J)>(x);
    if constexpr (J >= 2) slice_add<SL::at(J - 2), SL::at(J - 1)>(x, sum);
  }
  fence_sched();
  if constexpr (J + 1 < KS) rows_slots<F32, KS, J + 1, FOLD>(acc, qf, kf, x, c2, sum);
}

template <bool MAX>
__device__ __forceinline__ float both(float a, float b) { return MAX ? fmaxf(a, b) : a + b; }

// 16 values per lane over the 32 lanes of each half: the lane ends with the total of value lane / 2 % 16.
template <bool MAX>
__device__ __forceinline__ float half_totals(float (&c)[16], int lane) {
  auto perm = [](float v, auto ctrl) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), decltype(ctrl)::value, 0xf, 0xf, false));
  };
#pragma unroll
  for (int v = 0; v < 8; v++) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(c[v]), __float_as_uint(c[v + 8]), false, false);
    c[v] = both<MAX>(__uint_as_float(r[0]), __uint_as_float(r[1]));
  }
  auto halve = [&](auto count, int bit, auto ctrl) __attribute__((always_inline)) {
    constexpr int n = decltype(count)::value;
    const bool up = (lane & bit) != 0;
#pragma unroll
    for (int v = 0; v < n; v++) {
      const float keep = up ? c[v + n] : c[v], send = up ? c[v] : c[v + n];
      c[v] = both<MAX>(keep, perm(send, ctrl));
    }
  };
  halve(std::integral_constant<int, 4>{}, 8, std::integral_constant<int, 0x128>{});  // row_ror:8
  halve(std::integral_constant<int, 2>{}, 4, std::integral_constant<int, 0x141>{});  // row_half_mirror
  halve(std::integral_constant<int, 1>{}, 2, std::integral_constant<int, 0x4E>{});   // quad_perm [2,3,0,1]
  return both<MAX>(c[0], perm(c[0], std::integral_constant<int, 0xB1>{}));           // quad_perm [1,0,3,2]
}

// 1 / x to within an ulp, for x far from the ends of the range
__device__ __forceinline__ float inverse(float x) {
  const float r = __builtin_amdgcn_rcpf(x);
  return fmaf(fmaf(-x, r, 1.0f), r, r);
}

// T tiles of 32 keys per wave.  Accumulator layout as in score_mfma.hip, pass 2: a lane has one key column and 16 query rows.
// Workgroup `split` of a head takes its blocks of 32 rows split, split + splits, .. and writes their scores, or with several
// splits its part of them, to out + split * n_heads * N.
template <bool F32, int HD, int KS, bool EXACT, int T>
__global__ __launch_bounds__(kWaves * 64, 2) void score_rows(const bf16_t* __restrict__ q, const bf16_t* __restrict__ k,
                                                             float* __restrict__ out, KernelPlan pl, int splits) {
  using TL = Tile<HD>;
  constexpr int kKeyBytes = TL::kTileBytes / 2;  // 32 keys
  constexpr int kPerSlab = TL::kRowsPerSlab, kSlabs = 32 / kPerSlab;
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];  // [kWaves][2] tiles of 32 keys
  float* again = reinterpret_cast<float*>(smem + kWaves * TL::kTileBytes);  // [kWaves][T][64]
  __shared__ float part[kWaves][32];
  __shared__ __attribute__((aligned(16))) float refs[32], invs[32];
  __shared__ uint32_t odd;  // a bit per block of 32 rows, of which there are at most 8 (row_splits in launch_rules.h)
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int lane = threadIdx.x & 63, l32 = lane & 31, hi = lane >> 5;
  // the workgroups of a head read the same keys and go to one XCD: id = xcd + 8 * (split + splits * (bh / 8)), bh % 8 = xcd
  const int within = blockIdx.x >> 3;
  const int split = within % splits, bh = within / splits * 8 + (blockIdx.x & 7);
  if (bh >= pl.nb * pl.Hkv) return;
  const int b = batch_of(pl, bh), h = bh - b * pl.Hkv;
  clear_claims(pl, bh, split == 0);
  const int N = ctx_rows(pl, bh);
  if (N == 0) return;
  const int total = N + (pl.causal_patch ? pl.p : 0);
  const int blocks = (pl.R + 31) / 32, last_chunk = pl.d / 8 - 1;
  const float c2 = pl.c2;
  const bool is_max = pl.reduce == EPICACHE_REDUCE_MAX;
  const unsigned char* keys_of_head = reinterpret_cast<const unsigned char*>(k + b * pl.ksb + (int64_t)h * pl.ksh);
  const uint32_t kstride = (uint32_t)pl.kst * 2;
  const uint32_t my_keys = lds_address(smem) + wave * 2 * kKeyBytes;
  const unsigned char* my_lds = smem + wave * 2 * kKeyBytes;

  // Tile i of the wave is tile wave + kWaves * i of the head.  It goes through the wave's own part of LDS: no barrier.
  auto first_key = [&](int i) __attribute__((always_inline)) { return (wave + kWaves * i) * 32; };
  auto stage = [&](int i, int buf) __attribute__((always_inline)) {
    const int r0 = lane / TL::kChunks, c0 = lane % TL::kChunks;
    int first = first_key(i);
    const unsigned char* from = keys_of_head;
    uint32_t at = my_keys;
    // The addresses are made here and one from the other.  Made in advance they are spilled, and a load must not follow the lane
    // read that fetches its address too closely.
    asm volatile("" : "+s"(from), "+s"(first), "+s"(at));
    at += buf * kKeyBytes;
    if (EXACT && first + 32 <= total) {
      from += (size_t)first * kstride;
      const uint32_t row = r0 * kstride;
#pragma unroll
      for (int s = 0; s < kSlabs; s++) {
        asm volatile("" : "+s"(from), "+s"(at));
        dma16_uniform_base(at, from, row + ((c0 ^ TL::swz(s * kPerSlab + r0)) << 4));
        from += kPerSlab * kstride;
        at += 1024;
      }
    } else {
#pragma unroll
      for (int s = 0; s < kSlabs; s++) {
        asm volatile("" : "+s"(at));
        const int r = s * kPerSlab + r0, chunk = c0 ^ TL::swz(r);
        const unsigned char* mine = from + (size_t)min(first + r, total - 1) * kstride + min(chunk, last_chunk) * 16;
        if (!EXACT && chunk > last_chunk) mine = reinterpret_cast<const unsigned char*>(&kZeroChunk);
        dma16_lane_ptr(at, mine);
        at += 1024;
      }
    }
  };
  bf16x8 kf[KS], qf[KS];
  auto take = [&](int buf) __attribute__((always_inline)) {
    read_frags<HD, KS>(kf, my_lds + buf * kKeyBytes, 0, l32, hi);
#pragma unroll
    for (int j = 0; j < KS; j++) asm volatile("" : "+v"(kf[j]));
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): read before what comes next is written there
  };
  auto load_queries = [&](int block) __attribute__((always_inline)) {
    int g, t;
    head_and_token(pl.p, pl.inv_p, min(block * 32 + l32, pl.R - 1), g, t);
    load_row_frags<KS>(qf, q + b * pl.qsb + (int64_t)(h * pl.G + g) * pl.qsh + (int64_t)t * pl.qst, hi, pl.d);
  };
  // x of the rows that do not take key `first + l32` in becomes `out_of_sight`
  auto mask = [&](f32x16& x, int first, int block, float out_of_sight) __attribute__((always_inline)) {
    if (first + 32 <= N) return;
    const int key = first + l32;
#pragma unroll
    for (int v = 0; v < 16; v++) {
      bool seen = key < N;
      if (pl.causal_patch && key < total) {
        int g, t;
        head_and_token(pl.p, pl.inv_p, min(block * 32 + (v >> 2) * 8 + hi * 4 + (v & 3), pl.R - 1), g, t);
        seen = key - N <= t;
      }
      x[v] = seen ? x[v] : out_of_sight;
    }
  };
  // a value per row of the block, from all waves, in `to`
  auto rows_total = [&](auto max_c, float (&c)[16]) __attribute__((always_inline)) {
    const float mine = half_totals<decltype(max_c)::value>(c, lane);
    const int v = lane >> 1 & 15;
    if ((lane & 1) == 0) part[wave][(v >> 2) * 8 + hi * 4 + (v & 3)] = mine;
    __syncthreads();
    float t = 0.f;
    if (threadIdx.x < 32) {
      t = part[0][threadIdx.x];
#pragma unroll
      for (int w = 1; w < kWaves; w++) t = both<decltype(max_c)::value>(t, part[w][threadIdx.x]);
    }
    return t;
  };

  auto is_odd = [&](int block) __attribute__((always_inline)) {
    return (__builtin_amdgcn_readfirstlane(odd) >> block & 1) != 0;
  };

  float col[T];
#pragma unroll
  for (int i = 0; i < T; i++) col[i] = 0.f;
  if (threadIdx.x == 0) odd = 0;
  stage(0, 0);
  stage(1, 1);
  load_queries(split);
  int turn = 0;  // the buffer of the next block's first tile
#pragma unroll 1
  for (int block = split; block < blocks; block += splits) {
    const bool more = block + splits < blocks;
    asm volatile("" : "+v"(lane));  // what follows from it is made again in every round
    l32 = lane & 31, hi = lane >> 5;
    f32x16 x[T];
    float sum[16];
#pragma unroll
    for (int v = 0; v < 16; v++) sum[v] = 0.f;
    static_for<T>([&](auto i_c) __attribute__((always_inline)) {
      constexpr int i = decltype(i_c)::value, before = i > 0 ? i - 1 : 0;
      using SL = Slices<KS>;
      // the tile behind this one may still be on its way
      if (i + 1 < T || more) __builtin_amdgcn_s_waitcnt(0x0F70 | kSlabs);
      else wait_vmem();
      const int buf = T % 2 == 0 ? i & 1 : (i + turn) & 1;
      take(buf);
      if (i + 2 < T) stage(i + 2, buf);
      else if (more) stage(i + 2 - T, buf);
      rows_slots<F32, KS, 0, (i > 0)>(x[i], qf, kf, x[before], c2, sum);
      if constexpr (i > 0) {
        slice_exp<SL::at(KS - 1), SL::at(KS)>(x[before]);
        slice_add<SL::at(KS - 2), SL::at(KS)>(x[before], sum);
      }
    });
    turn ^= 1;
    slice_scale<0, 16>(x[T - 1], c2);
    slice_exp<0, 16>(x[T - 1]);
    // masked tiles are the wave's last ones: their sums are made again
    if (first_key(T - 1) + 32 > N) {
#pragma unroll
      for (int v = 0; v < 16; v++) sum[v] = 0.f;
      static_for<T>([&](auto i_c) __attribute__((always_inline)) {
        constexpr int i = decltype(i_c)::value;
        mask(x[i], first_key(i), block, 0.f);
        slice_add<0, 16>(x[i], sum);
      });
    } else {
      slice_add<0, 16>(x[T - 1], sum);
    }
    const float rows = rows_total(std::false_type{}, sum);
    if (threadIdx.x < 32) {
      const bool row = block * 32 + (int)threadIdx.x < pl.R;
      invs[threadIdx.x] = row ? inverse(rows) : 0.f;
      if (row && !(rows <= kMostTotal && rows >= kLeastTotal)) atomicOr(&odd, 1u << block);
    }
    if (more) load_queries(block + splits);
    __syncthreads();
    if (is_odd(block)) continue;
    float inv[16];
#pragma unroll
    for (int g4 = 0; g4 < 4; g4++) {
      const float4 a = *reinterpret_cast<const float4*>(invs + g4 * 8 + hi * 4);
      inv[g4 * 4 + 0] = a.x, inv[g4 * 4 + 1] = a.y, inv[g4 * 4 + 2] = a.z, inv[g4 * 4 + 3] = a.w;
    }
    static_for<T>([&](auto i_c) __attribute__((always_inline)) {
      constexpr int i = decltype(i_c)::value;
      if (is_max) {
#pragma unroll
        for (int v = 0; v < 16; v++) col[i] = fmaxf(col[i], x[i][v] * inv[v]);
      } else {
        float s0 = 0.f, s1 = 0.f;
#pragma unroll
        for (int v = 0; v < 16; v += 2) s0 = fmaf(x[i][v], inv[v], s0), s1 = fmaf(x[i][v + 1], inv[v + 1], s1);
        col[i] += s0 + s1;
      }
    });
  }
  // Blocks with odd rows, one tile at a time, three times over: the rows' maxima, their sums, the weights.
#pragma unroll 1
  for (int block = split; block < blocks; block += splits) {
    if (!is_odd(block)) continue;
    load_queries(block);
#pragma unroll 1
    for (int pass = 0; pass < 3; pass++) {
      float acc[16];
#pragma unroll
      for (int v = 0; v < 16; v++) acc[v] = pass == 0 ? kNoMax : 0.f;
#pragma unroll 1
      for (int i = 0; i < T; i++) {
        asm volatile("" : "+v"(lane));
        l32 = lane & 31, hi = lane >> 5;
        stage(i, 0);
        wait_vmem();
        take(0);
        f32x16 y;
        mfma_chain<KS, F32>(y, qf, kf);
        mask(y, first_key(i), block, kMasked);
        float c = 0.f;
        const volatile float *ref = refs + hi * 4, *inv = invs + hi * 4;
#pragma unroll
        for (int v = 0; v < 16; v++) {
          if (pass == 0) {
            acc[v] = fmaxf(acc[v], y[v]);
          } else {
            const float e = ex2(fmaf(y[v], c2, -ref[(v >> 2) * 8 + (v & 3)]));
            if (pass == 1) acc[v] += e;
            else c = is_max ? fmaxf(c, e * inv[(v >> 2) * 8 + (v & 3)]) : fmaf(e, inv[(v >> 2) * 8 + (v & 3)], c);
          }
        }
        if (pass == 2) again[(wave * T + i) * 64 + lane] = c;
      }
      if (pass == 2) break;
      const float rows = pass == 0 ? rows_total(std::true_type{}, acc) : rows_total(std::false_type{}, acc);
      if (threadIdx.x < 32) {
        if (pass == 0) refs[threadIdx.x] = rows * c2;
        else invs[threadIdx.x] = block * 32 + (int)threadIdx.x < pl.R ? inverse(rows) : 0.f;
      }
      __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < T; i++) {
      const float more = again[(wave * T + i) * 64 + lane];
      col[i] = is_max ? fmaxf(col[i], more) : col[i] + more;
    }
  }
  float* row = out + ((size_t)split * (pl.nb * pl.Hkv) + bh) * pl.N;
#pragma unroll
  for (int i = 0; i < T; i++) {
    // lanes l and l^32 hold the same key over disjoint rows
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(col[i]), __float_as_uint(col[i]), false, false);
    const float lo = __uint_as_float(r[0]), up = __uint_as_float(r[1]);
    const int key = first_key(i) + l32;
    if (hi == 0 && key < N) row[key] = is_max ? fmaxf(lo, up) : lo + up;
  }
}

// The parts of several workgroups of a head, in order.
__global__ void merge_rows(const float* __restrict__ parts, float* __restrict__ scores, size_t n, int splits, int is_max) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  float x = parts[i];
  for (int s = 1; s < splits; s++) x = is_max ? fmaxf(x, parts[s * n + i]) : x + parts[s * n + i];
  scores[i] = x;
}

template <bool F32, int HD, int KS, bool EXACT, int T>
hipError_t launch_tiles(const Plan& pl, const bf16_t* q, const bf16_t* k, float* out, hipStream_t stream) {
  const size_t smem = kWaves * (Tile<HD>::kTileBytes + T * 64 * sizeof(float));
  auto kernel = score_rows<F32, HD, KS, EXACT, T>;
  if (smem > 64 * 1024) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
    if (e != hipSuccess) return e;
  }
  const int heads = pl.nb * pl.Hkv;
  hipLaunchKernelGGL(kernel, dim3((heads + 7) / 8 * 8 * pl.row_splits), dim3(kWaves * 64), smem, stream, q, k, out, pl, pl.row_splits);
  return hipGetLastError();
}

template <bool F32, int HD, int KS, bool EXACT, int T = kFewestTiles>
hipError_t launch_rows(const Plan& pl, const bf16_t* q, const bf16_t* k, float* out, hipStream_t stream) {
  const int keys = pl.N + (pl.causal_patch ? pl.p : 0);
  if constexpr (T < kMostTiles)
    if (keys > T * kWaves * 32) return launch_rows<F32, HD, KS, EXACT, T + 1>(pl, q, k, out, stream);
  return launch_tiles<F32, HD, KS, EXACT, T>(pl, q, k, out, stream);
}

}  // namespace

hipError_t launch_score_rows(const Plan& pl, const void* q, const void* k, float* scores, hipStream_t stream) {
  const bf16_t* qq = static_cast<const bf16_t*>(q);
  const bf16_t* kk = static_cast<const bf16_t*>(k);
  float* out = pl.row_splits > 1 ? pl.score_parts : scores;
  hipError_t e;
  if (pl.dtype == EPICACHE_DTYPE_F32) {
    Plan p2 = pl;  // fp32 rows are moved as rows of twice as many two-byte units
    p2.d *= 2;
    for (int64_t* s : {&p2.qsb, &p2.qsh, &p2.qst, &p2.ksb, &p2.ksh, &p2.kst}) *s *= 2;
    e = launch_rows<true, 128, 8, true>(p2, qq, kk, out, stream);
  } else if (pl.d == 64) {
    e = launch_rows<false, 64, 4, true>(pl, qq, kk, out, stream);
  } else if (pl.d == 128) {
    e = launch_rows<false, 128, 8, true>(pl, qq, kk, out, stream);
  } else {
    e = launch_rows<false, 128, 6, false>(pl, qq, kk, out, stream);
  }
  if (e != hipSuccess || pl.row_splits == 1 || !scores) return e;
  const size_t n = (size_t)pl.nb * pl.Hkv * pl.N;
  hipLaunchKernelGGL(merge_rows, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream, pl.score_parts, scores, n, pl.row_splits,
                     (int)(pl.reduce == EPICACHE_REDUCE_MAX));
  return hipGetLastError();
}

}  // namespace epicache

// Per-(batch item, KV head) top-M selection (the retention rule of paper Sec. 3.1
// Stage 2 / Alg. 1 phase A3), exact.
//
// One workgroup owns one score row and holds it in registers as unsigned keys whose integer order is the float
// order (select_util.h has the search and the emission).  Kept: all keys above the n_keep-th largest, plus the first
// ones equal to it (lower index wins a tie), which makes the count exactly n_keep and keeps the output ascending.
#include "epicache_internal.h"
#include "select_util.h"

namespace epicache {
namespace {

// Keys in registers, VPT per thread (N <= NW * 64 * VPT).
template <int VPT, int NW>
__global__ __launch_bounds__(NW * 64, VPT <= 24 ? 8 : 4) void topk_select(const float* __restrict__ scores, int32_t* __restrict__ keep,
                                                       int N, int n_keep, int pitch, int appended) {
  __shared__ SelectLds<NW> sm;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const float* row = scores + (size_t)blockIdx.x * N;
  const int base = wave * VPT * 64 + lane;
  uint32_t keys[VPT], least;
  load_keys(keys, least, row, base, N);
  const Threshold t = select_threshold<VPT, NW>(keys, least, N, (uint32_t)n_keep, wave, lane, sm);
  int32_t* out = keep + (size_t)blockIdx.x * pitch;  // rows of kept indices are `pitch` apart
  emit_kept<VPT, NW>(keys, base, N, t, IntoRow{out, (uint32_t)n_keep}, wave, 0, lane, sm);
  for (int i = tid; i < appended; i += NW * 64) out[n_keep + i] = N + i;  // rows kept whatever they score
}

// Rows too long for the registers: keys are re-read from global memory, so the sweeps are few (four 8-bit histogram
// digits, most significant first) instead of many cheap ones.
__global__ __launch_bounds__(1024) void topk_select_long(const float* __restrict__ scores,
                                                         int32_t* __restrict__ keep, int N, int n_keep,
                                                         int pitch, int appended) {
  __shared__ uint32_t hist_rep[256 * kHistCopies];  // one digit's histogram, every bin once per LDS bank
  __shared__ uint32_t hist[256];
  __shared__ uint32_t wave_gt[16], wave_eq[16];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int nwaves = blockDim.x >> 6;
  const float* row = scores + (size_t)blockIdx.x * N;
  int32_t* out = keep + (size_t)blockIdx.x * pitch;  // rows of kept indices are `pitch` apart

  const int groups = (N + nwaves * 64 - 1) / (nwaves * 64);  // 64-wide groups per wave
  const int base = wave * groups * 64 + lane;
  auto key_at = [&](int j) -> uint32_t {
    const int i = base + j * 64;
    return i < N ? order_key(row[i]) : 0u;
  };

  for (int i = tid; i < 256 * kHistCopies; i += blockDim.x) hist_rep[i] = 0;
  __syncthreads();

  uint32_t prefix = 0, mask = 0;
  uint32_t kth = (uint32_t)n_keep;  // rank (1 = largest) still to be located inside the current prefix class
#pragma unroll 1
  for (int pass = 0; pass < 4; pass++) {
    const int shift = 24 - 8 * pass;
    for (int j = 0; j < groups; j++) {
      const uint32_t key = key_at(j);
      if (base + j * 64 < N && (key & mask) == prefix) hist_count(hist_rep, (key >> shift) & 255u, lane);
    }
    __syncthreads();
    hist_fold(hist_rep, hist, tid);
    __syncthreads();
    uint32_t bin, above;
    locate_digit(hist, kth, lane, bin, above);  // every wave scans the 256 bins itself
    prefix |= bin << shift;
    mask |= 255u << shift;
    kth -= above;
  }
  const uint32_t thr = prefix;    // key of the n_keep-th largest score
  const uint32_t need_eq = kth;   // how many keys equal to thr are kept (>= 1)

  // per-wave counts, then an exclusive prefix over the waves
  uint32_t cgt = 0, ceq = 0;
  for (int j = 0; j < groups; j++) {
    const uint32_t key = key_at(j);
    const bool valid = base + j * 64 < N;
    cgt += __popcll(__ballot(valid && key > thr));
    ceq += __popcll(__ballot(valid && key == thr));
  }
  if (lane == 0) wave_gt[wave] = cgt, wave_eq[wave] = ceq;
  __syncthreads();
  uint32_t gt_before = 0, eq_before = 0;
  for (int w = 0; w < wave; w++) gt_before += wave_gt[w], eq_before += wave_eq[w];

  for (int j = 0; j < groups; j++) {
    const uint32_t key = key_at(j);
    const int i = base + j * 64;
    const bool valid = i < N;
    const bool is_gt = valid && key > thr, is_eq = valid && key == thr;
    const uint64_t bgt = __ballot(is_gt), beq = __ballot(is_eq);
    const uint32_t my_gt = gt_before + lanes_below(bgt);
    const uint32_t my_eq = eq_before + lanes_below(beq);
    if (is_gt || (is_eq && my_eq < need_eq)) out[my_gt + min(my_eq, need_eq)] = i;
    gt_before += __popcll(bgt);
    eq_before += __popcll(beq);
  }
  for (int i = tid; i < appended; i += blockDim.x) out[n_keep + i] = N + i;
}

__global__ void iota_keep(int32_t* keep, int n_keep, size_t total) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < total) keep[i] = (int32_t)(i % n_keep);
}

}  // namespace

hipError_t launch_iota_keep(const Plan& pl, int32_t* keep, hipStream_t stream) {
  const size_t total = (size_t)pl.nb * pl.Hkv * pl.n_keep;
  hipLaunchKernelGGL(iota_keep, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, stream, keep,
                     pl.n_keep, total);
  return hipGetLastError();
}

hipError_t launch_topk(const Plan& pl, const float* scores, int32_t* keep, int appended, hipStream_t stream) {
  if (pl.N <= pl.M) return launch_iota_keep(pl, keep, stream);
  const int nbh = pl.nb * pl.Hkv, N = pl.N, nk = pl.n_keep, pitch = pl.keep_stride;
  auto launch = [&](auto kernel, int nw) {
    hipLaunchKernelGGL(kernel, dim3(nbh), dim3(nw * 64), 0, stream, scores, keep, N, nk, pitch, appended);
  };
  // Waves per row (kernel time, 32 rows / 512 rows / 896 rows): N = 512 in 4 waves 4.3 / 4.6 us, in 8 4.6 / 5.2; 2048 in 4 5.2 /
  // 6.4, in 8 4.6 / 7.0; 4096 in 4 6.4 / 9.2 / 12.3, in 8 5.7 / 9.3 / 15.4, in 16 6.6 / 11.3; 8192 in 4 10.8 / 15.2, in 8 8.4 /
  // 13.7, in 16 8.7 / 15.4.
  const bool few = nbh <= 256;
  if (N <= 1024) launch(topk_select<4, 4>, 4);
  else if (N <= 2048) few ? launch(topk_select<4, 8>, 8) : launch(topk_select<8, 4>, 4);
  else if (N <= 4096) few ? launch(topk_select<8, 8>, 8) : launch(topk_select<16, 4>, 4);
  else if (N <= 8192) launch(topk_select<16, 8>, 8);
  else if (N <= 16384) launch(topk_select<16, 16>, 16);
  else if (N <= 24576) launch(topk_select<24, 16>, 16);
  else if (N <= 32768) launch(topk_select<32, 16>, 16);
  else launch(topk_select_long, 16);
  return hipGetLastError();
}

}  // namespace epicache

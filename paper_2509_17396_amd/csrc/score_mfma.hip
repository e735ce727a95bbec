// MFMA scoring kernels for gfx950: bf16 of any head_dim up to 256, fp32 up to 128 (multiples of 8).
//
// Eq. 1 needs every row's softmax normaliser over all N context keys before a
// single column value is final, and the R x N logits of one KV head do not fit
// on chip, so Q.K^T is evaluated twice:
//   pass 1 (score_stats):  per query row, a reference logit (the maximum, or a value
//                          within 2^60 in weight of it) and the sum of exp2 relative
//                          to it over the keys of one key split -> stats[bh][split][row]
//   pass 2 (score_reduce): per context key, reduce exp2(logit - lse_row) over
//                          all R = G*p rows (max or sum) -> scores[bh][key]
// Both use v_mfma_f32_32x32x16_bf16 (or, on fp32 inputs, v_mfma_f32_32x32x2_f32) with fp32 accumulation.  The operand order
// is chosen so that the axis being reduced lies inside a lane's 16 accumulator
// values: pass 1 puts the keys on the MFMA row axis (a lane owns one query
// column and 16 keys), pass 2 puts the query rows there (a lane owns one key
// column and 16 query rows).  Only two lanes (l, l^32) ever need to be combined.
//
// Both passes are bound by the plain ALUs, not by the matrix cores: per logit
// the softmax costs a multiply-add, an exponential (half rate) and an add or
// max, about 4 issue slots, against 2 slots' worth of MFMA time.  Each wave
// therefore software-pipelines by hand: the MFMA chain of tile u+1 is issued
// one instruction at a time between slices of the softmax arithmetic of tile u.
//
// Accumulator layout of the 32x32 MFMA: lane l, value v holds
//   row = (v / 4) * 8 + (l / 32) * 4 + (v % 4),  column = l % 32.
// The contraction index a lane feeds is the same for the A and the B operand
// (16-byte chunk 2*j + l/32 of the head_dim row for MFMA j), which is all the
// hardware needs for a correct dot product.
//
// Staging: 64-row tiles (keys in pass 1, query rows in pass 2) go from global
// memory straight into LDS with global_load_lds_dwordx4 (lane l of a wave fills
// 16-byte slot l of a 1 KiB slab).  Each lane picks the global chunk that makes
// the LDS image XOR-swizzled, so the ds_read_b128 of the MFMA operands is free
// of bank conflicts without padding.
#include <type_traits>

#include "epicache_internal.h"
#include "launch_rules.h"
#include "mfma_tiles.h"

namespace epicache {
namespace {

// Form of the rows, and of what pass 2 knows about a row's normaliser:
//   kFolded  bf16 rows of exactly 64 or 128 elements: one number, the row's base-2 log-sum-exp, added to every logit.
//            Rounded at the size of the logits, it costs a weight up to 2^-24 |lse| of its value.
//   kBf16    bf16 rows of any other length up to 256, kF32: fp32 rows of up to 128.  The reference and the sum of pass 1
//            apart: a weight is exp2(logit - reference) * (1 / sum), as exact as a division per weight.  Errors against
//            float64, relative, mean over keys (fp32, d = 64, logits of about 1; sum / max): folded 2.1e-7 / 3.9e-7,
//            apart 5.0e-8 / 2.6e-7.
enum Form { kFolded, kBf16, kF32 };

// ------------------------------------------------------------------ pass 1
// Softmax statistics of the previous accumulator tile, cut into slices that are
// issued between the MFMAs of the next tile.  16 values = 16 keys of one query row.
//
// Sentinels instead of infinities, so that no inf - inf can arise: a row that has
// seen no key yet has m = kNoMax; masked keys and the filler tile that precedes the
// first real one hold kMasked < kNoMax, so folding them in leaves (m, D) untouched
// (their exp2 underflows to exactly 0 and the max does not move).  Raw dot products
// are assumed to lie above kNoMax (-1e30).
struct RowStat {
  float m, D;  // reference (a raw dot product at or below the running maximum); running sum of exp2((dot - m) * c2)
};

// Factor that takes a sum from the reference `from` to the reference `to`.  Sums are relative to exp2 of the rounded
// product reference * c2, so where the errors count the exponent is the difference of two such numbers (pinned: contracted
// into the difference, a product would go in unrounded); both give exactly 1 where the reference did not move.
template <int FORM>
__device__ __forceinline__ float correction(float from, float to, float c2) {
  if (FORM == kFolded) return ex2((from - to) * c2);
  float x = from * c2, y = to * c2;
  pin(x), pin(y);
  return ex2(x - y);
}

template <int FORM>
__device__ __forceinline__ void stats_begin(const f32x16& P, const RowStat& st, float c2, float& mn,
                                            float& nmc, float& corr) {
  const float a0 = max3(P[0], P[1], P[2]), a1 = max3(P[3], P[4], P[5]), a2 = max3(P[6], P[7], P[8]);
  const float a3 = max3(P[9], P[10], P[11]), a4 = max3(P[12], P[13], P[14]);
  mn = max3(max3(a0, a1, a2), max3(a3, a4, P[15]), st.m);
  nmc = -mn * c2;
  corr = correction<FORM>(st.m, mn, c2);
}

// Which accumulator values enter the arithmetic pipeline in each MFMA slot of a unit.  Independent vector
// instructions issue in the shadow of an MFMA, so the softmax arithmetic is spread evenly over the KS slots;
// and because dependent VALU / transcendental ops have several clocks of latency, it is staggered: the
// values that get their multiply-add in slot j get their exp2 in slot j+1 and are summed in slot j+2, so
// the instructions inside one slot never wait on each other.
template <int KS> struct Slots {  // KS MFMAs, KS in {2, 4, 6, 8, 12, 16}
  static constexpr int reduce(int j) { return KS == 6 ? (j < 5 ? 3 * j : j == 5 ? 14 : 16) : (16 * j) / KS; }
};

// pipeline stages over the value range [LO, HI); each pins its results at the point of issue
template <int LO, int HI>
__device__ __forceinline__ void stage_exp(float (&x)[16]) {
#pragma unroll
  for (int v = LO; v < HI; v++) x[v] = ex2(x[v]);
#pragma unroll
  for (int v = LO; v < HI; v++) pin(x[v]);
}
template <int LO, int HI>
__device__ __forceinline__ void stage_add(const float (&x)[16], float& s0, float& s1) {
#pragma unroll
  for (int v = LO; v < HI; v++) {
    if (v & 1) s1 += x[v]; else s0 += x[v];
  }
  if (HI > LO) pin(s0), pin(s1);
}
template <int LO, int HI>
__device__ __forceinline__ void stage_max(const float (&x)[16], float& s0, float& s1) {
#pragma unroll
  for (int v = LO; v < HI; v += 2) {  // two values per instruction, alternating between the two chains
    float& s = ((v - LO) & 2) ? s1 : s0;
    if (v + 1 < HI) s = vmax3(s, x[v], x[v + 1]);
    else s = vmax(s, x[v]);
  }
  if (HI > LO) pin(s0), pin(s1);
}

template <int LO, int HI>
__device__ __forceinline__ void stats_stage_fma(float (&x)[16], const f32x16& P, float c2, float nmc) {
#pragma unroll
  for (int v = LO; v < HI; v++) x[v] = fmaf(P[v], c2, nmc);
#pragma unroll
  for (int v = LO; v < HI; v++) pin(x[v]);
}

__device__ __forceinline__ float stats_group(const f32x16& P, int g, float c2, float nmc) {
  const float e0 = ex2(fmaf(P[4 * g + 0], c2, nmc)), e1 = ex2(fmaf(P[4 * g + 1], c2, nmc));
  const float e2 = ex2(fmaf(P[4 * g + 2], c2, nmc)), e3 = ex2(fmaf(P[4 * g + 3], c2, nmc));
  return (e0 + e1) + (e2 + e3);
}

// acc <- MFMA chain over head_dim (A rows = a-frag rows, B columns = b-frag rows), interleaved
// with folding P, the tile finished one unit earlier, into its row statistics.
// The reference st.m of a row only has to keep the exponentials in range, so the fast path does not look
// for the tile's maximum at all (12 of ~62 instructions per unit): it sums exp2((dot - st.m) * c2) as is and
// checks the sum.  A sum beyond kRebase (a dot product more than ~60 / c2 above the reference, or a row
// that has no reference yet: st.m = kNoMax sends every real dot product to +inf) takes the exact path
// below, which moves the reference to the true maximum.  Wave-uniform branch, taken for the first tile of
// a row and then only when the logits climb by a factor of 2^60 in weight.
// Where the errors of a weight count (other than kFolded) the reference stays closer: a key that is x above it in the
// exponent enters with x rounded, and differently in the two passes.  There the 16 keys of a unit may sum up to 2^16, so
// that x stays below 16 and its rounding below 2^-21.
constexpr float kRebase = 1.0e18f;
constexpr float kRebaseUnit = 65536.f;

template <int FORM, int KS, int J>
__device__ __forceinline__ void stats_slot(f32x16& acc, const bf16x8 (&a)[KS], const bf16x8 (&b)[KS],
                                           const f32x16& P, float c2, float nmc, float (&x)[16], float& s0,
                                           float& s1) {
  using SL = Slots<KS>;
  if (J == 0) acc = f32x16{0};
  mfma_step<FORM == kF32>(acc, a[J], b[J]);
  fence_sched();
  stats_stage_fma<SL::reduce(J), SL::reduce(J + 1)>(x, P, c2, nmc);
  if constexpr (J >= 1) stage_exp<SL::reduce(J - 1), SL::reduce(J)>(x);
  if constexpr (J >= 2) stage_add<SL::reduce(J - 2), SL::reduce(J - 1)>(x, s0, s1);
  fence_sched();
}

template <int FORM, int KS, int J = 0>
__device__ __forceinline__ void stats_slots(f32x16& acc, const bf16x8 (&a)[KS], const bf16x8 (&b)[KS],
                                            const f32x16& P, float c2, float nmc, float (&x)[16], float& s0,
                                            float& s1) {
  stats_slot<FORM, KS, J>(acc, a, b, P, c2, nmc, x, s0, s1);
  if constexpr (J + 1 < KS) stats_slots<FORM, KS, J + 1>(acc, a, b, P, c2, nmc, x, s0, s1);
}

template <int FORM>
__device__ __forceinline__ void stats_fold(const f32x16& P, RowStat& st, float c2);

// DEFER: the sum is taken as it is and only the largest one of several units is kept in `worst`; the
// caller checks that once per key tile and, if it ever exceeded the limit, redoes those units on the exact path.
template <int FORM, int KS, bool DEFER = false>
__device__ __forceinline__ void stats_unit(f32x16& acc, const bf16x8 (&a)[KS], const bf16x8 (&b)[KS],
                                           const f32x16& P, RowStat& st, float c2, float* worst = nullptr) {
  using SL = Slots<KS>;
  float s0 = 0.f, s1 = 0.f, x[16];
  const float nmc = -st.m * c2;
  stats_slots<FORM, KS>(acc, a, b, P, c2, nmc, x, s0, s1);
  // drain the pipeline: last exp2 stage, last two sum stages
  stage_exp<SL::reduce(KS - 1), SL::reduce(KS)>(x);
  stage_add<SL::reduce(KS - 2), SL::reduce(KS - 1)>(x, s0, s1);
  stage_add<SL::reduce(KS - 1), SL::reduce(KS)>(x, s0, s1);
  const float D = st.D + (s0 + s1);
  const float checked = FORM == kFolded ? D : s0 + s1;
  constexpr float kLimit = FORM == kFolded ? kRebase : kRebaseUnit;
  if constexpr (DEFER) {
    st.D = D;  // +inf at worst (a row without a reference, or a logit 2^60 in weight above it): never NaN
    *worst = fmaxf(*worst, checked);
  } else {
    if (__any(!(checked <= kLimit))) stats_fold<FORM>(P, st, c2);  // some row needs a new reference: exact path for the wave
    else st.D = D;
  }
  fence_sched();
}

// fold one finished tile into its row statistics, nothing to overlap with
template <int FORM>
__device__ __forceinline__ void stats_fold(const f32x16& P, RowStat& st, float c2) {
  float mn, nmc, corr;
  stats_begin<FORM>(P, st, c2, mn, nmc, corr);
  const float s = (stats_group(P, 0, c2, nmc) + stats_group(P, 1, c2, nmc)) +
                  (stats_group(P, 2, c2, nmc) + stats_group(P, 3, c2, nmc));
  st.D = fmaf(st.D, corr, s);
  st.m = mn;
}

// Key tiles per split.  Where the heads have lengths of their own, often far below the bound that the plan was made
// for, every split takes its share of the head's own tiles; cut at the bound, the last splits were empty and part of
// the chip idle (64 heads of 7000 to 9000 of 13000 rows, R = 448: pass 1 97 -> 79 us).
__device__ __forceinline__ int split_length(const Plan& pl, int tiles, int splits, int tiles_per_split) {
  return pl.n_ctx ? __builtin_amdgcn_readfirstlane((tiles + splits - 1) / splits) : tiles_per_split;
}

// Head and part of the id-th of all heads' `parts` parts.
__device__ __forceinline__ void spread_parts(int id, int parts, int& bh, int& part) {
  bh = id / parts;
  part = id - bh * parts;
}

// NQ 32-row query sub-tiles per wave, NW waves per workgroup: 32*NQ*NW query rows per workgroup.
template <int FORM, int HD, int KS, int NQ, int NW>
__global__ __launch_bounds__(NW * 64, (NW == 1 || (HD > 128 && NW < 4) ? 1 : 2)) void score_stats(const bf16_t* __restrict__ q,
                                                          const bf16_t* __restrict__ k,
                                                          float2* __restrict__ stats, Plan pl) {
  using TL = Tile<HD>;
  using ST = Stager<HD, KS, NW, FORM == kFolded>;
  // the per-unit check of the running sums is deferred to once per tile where the registers allow it (the
  // three-sub-tile form sits at the 256-register limit as it is)
  constexpr bool kDeferCheck = NQ <= 2;
  __shared__ __attribute__((aligned(1024))) unsigned char lds[2 * TL::kTileBytes];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, hi = lane >> 5;
  // Workgroups are handed to the 8 XCDs round-robin by linear id.  The key splits (and row blocks) of one
  // (b, h) read the same query rows, so they are given ids that land on one XCD and share its L2:
  // id = xcd + 8 * (rb + RB * (split + S * (bh / 8))), bh % 8 = xcd; row blocks of a split side by side: one K fetch.
  const int rb = blockIdx.x >> 3;
  int split = blockIdx.y, bh = blockIdx.z * 8 + (blockIdx.x & 7);
  if (pl.spread) spread_parts(blockIdx.y * 8 + (blockIdx.x & 7), pl.n_splits, bh, split);
  if (bh >= pl.nb * pl.Hkv) return;
  const int b = batch_of(pl, bh), h = bh - b * pl.Hkv;
  const int row0 = rb * (32 * NQ * NW) + wave * (32 * NQ);
  const bool active = row0 < pl.R;  // waves without rows only help staging the key tiles
  const float c2 = pl.c2;

  const int N = ctx_rows(pl, bh);
  const int tiles = (N + kKeyTile - 1) / kKeyTile;
  const int tiles_per_split = split_length(pl, tiles, pl.n_splits, pl.tiles_per_split);
  const int t_begin = split * tiles_per_split;
  if (t_begin >= tiles) {
    // a head shorter than the batch's longest: this split holds none of its keys and contributes
    // an empty sum under a maximum below every logit
    const int r_end = min(pl.R, (rb + 1) * (32 * NQ * NW));
    for (int r = rb * (32 * NQ * NW) + tid; r < r_end; r += NW * 64)
      stats[((size_t)bh * pl.n_splits + split) * pl.Rpad + r] = make_float2(kMasked, 0.f);
    return;
  }
  const int t_end = min(tiles, t_begin + tiles_per_split);
  // a ragged last tile (N % 64 != 0) is handled after the pipelined loop over full tiles
  const int t_full = (t_end == tiles && N % kKeyTile != 0) ? t_end - 1 : t_end;

  // query fragments stay in registers for the whole key loop; rows beyond R repeat the last one, nothing reads theirs
  bf16x8 qf[NQ][KS];
#pragma unroll
  for (int s = 0; s < NQ; s++) {
    int g, t;
    head_and_token(pl.p, pl.inv_p, min(row0 + s * 32 + l32, pl.R - 1), g, t);
    load_row_frags<KS>(qf[s], q + b * pl.qsb + (int64_t)(h * pl.G + g) * pl.qsh + (int64_t)t * pl.qst, hi, pl.d);
  }

  const unsigned char* kbase = reinterpret_cast<const unsigned char*>(k + b * pl.ksb + (int64_t)h * pl.ksh);
  const uint32_t kstride = (uint32_t)pl.kst * 2;
  const int last_chunk = pl.d / 8 - 1;
  const typename ST::Offsets koff = ST::offsets(wave, lane, kstride, last_chunk);

  RowStat st[NQ];
#pragma unroll
  for (int s = 0; s < NQ; s++) st[s].m = kNoMax, st[s].D = 0.f;
  f32x16 accA, accB;
#pragma unroll
  for (int v = 0; v < 16; v++) accA[v] = accB[v] = kMasked;  // the tile "before the first": a no-op

  // in registers before the loop: a scalar load pending there makes every wait for an LDS read in it a wait for all
  int causal_patch = pl.causal_patch, Rpad = pl.Rpad, n_splits = pl.n_splits;
  float2* out = stats;
  asm volatile("" : "+s"(causal_patch), "+s"(Rpad), "+s"(n_splits), "+s"(out));
  const uint32_t lds0 = lds_address(lds);
  if (t_begin < t_full) ST::run(lds0, kbase + (size_t)t_begin * kKeyTile * kstride, koff, wave);
  wait_vmem();
  __syncthreads();
  int buf = 0;
  // Units of one tile, in order: (ks, s) for key half ks in {0,1}, query sub-tile s in 0..NQ-1.
  // Unit u accumulates into accA (u even) or accB (u odd) while unit u-1 is folded into the
  // statistics of its query sub-tile.  2*NQ is even, so the parity carries over between tiles.
  int t = t_begin;
  if (kDeferCheck && t < t_full) {
    // The rows have no reference yet, so the first tile goes through the exact path: all units but the last, which
    // is left in accB for the next tile.
    if (t + 1 < t_full) ST::run(lds0 + TL::kTileBytes, kbase + (size_t)(t + 1) * kKeyTile * kstride, koff, wave);
    if (active) {
      bf16x8 kf[KS];
#pragma unroll
      for (int u = 0; u < 2 * NQ - 1; u++) {
        if (u == 0 || u == NQ) read_frags<HD, KS>(kf, lds, u / NQ, l32, hi);
        mfma_chain<KS, FORM == kF32>(accA, kf, qf[u % NQ]);
        stats_fold<FORM>(accA, st[u % NQ], c2);
      }
      if (NQ == 1) read_frags<HD, KS>(kf, lds, 1, l32, hi);
      mfma_chain<KS, FORM == kF32>(accB, kf, qf[NQ - 1]);
    }
    wait_vmem();
    __syncthreads();
    buf = 1;
    t++;
  }
  for (; t < t_full; t++) {
    const unsigned char* cur = lds + buf * TL::kTileBytes;
    if (t + 1 < t_full)
      ST::run(lds0 + (buf ^ 1) * TL::kTileBytes, kbase + (size_t)(t + 1) * kKeyTile * kstride, koff, wave);
    if (active) {
      bf16x8 kf[KS];  // one 32-key half at a time, refilled once its last MFMA has been issued
      read_frags<HD, KS>(kf, cur, 0, l32, hi);
      if constexpr (kDeferCheck) {
        // The unit carried over from the previous tile is folded with its check at once (its keys are gone from
        // LDS).  The tile's own units 0 .. 2*NQ-2 are folded unchecked; one look at their largest sum decides
        // whether they are redone, from the row statistics as they were before them, on the exact path.  The
        // tile is still in LDS then, and neither kf nor accA is live any more.
        stats_unit<FORM, KS>(accA, kf, qf[0], accB, st[NQ - 1], c2);
        RowStat before[NQ];
#pragma unroll
        for (int s = 0; s < NQ; s++) before[s] = st[s];
        float worst = 0.f;
#pragma unroll
        for (int u = 1; u < 2 * NQ; u++) {
          const int s = u % NQ, sp = (u - 1) % NQ;
          if (u == NQ) read_frags<HD, KS>(kf, cur, 1, l32, hi);
          if (u & 1) stats_unit<FORM, KS, true>(accB, kf, qf[s], accA, st[sp], c2, &worst);
          else       stats_unit<FORM, KS, true>(accA, kf, qf[s], accB, st[sp], c2, &worst);
        }
        if (__any(!(worst <= (FORM == kFolded ? kRebase : kRebaseUnit)))) {
#pragma unroll
          for (int s = 0; s < NQ; s++) st[s] = before[s];
#pragma unroll
          for (int u = 0; u < 2 * NQ - 1; u++) {
            if (u == 0 || u == NQ) read_frags<HD, KS>(kf, cur, u / NQ, l32, hi);
            mfma_chain<KS, FORM == kF32>(accA, kf, qf[u % NQ]);
            stats_fold<FORM>(accA, st[u % NQ], c2);
          }
        }
      } else {
#pragma unroll
        for (int u = 0; u < 2 * NQ; u++) {
          const int s = u % NQ, sp = (u + NQ * 2 - 1) % NQ;
          if (u == NQ) read_frags<HD, KS>(kf, cur, 1, l32, hi);
          if (u & 1) stats_unit<FORM, KS>(accB, kf, qf[s], accA, st[sp], c2);
          else       stats_unit<FORM, KS>(accA, kf, qf[s], accB, st[sp], c2);
        }
      }
    }
    wait_vmem();
    __syncthreads();
    buf ^= 1;
  }
  if (active) stats_fold<FORM>(accB, st[NQ - 1], c2);  // last unit in flight (or the filler)

  if (t_full < t_end) {
    // ragged last tile: rows beyond N re-read the last key and are masked out of the statistics
    const int t = t_full;
    const int nrows = N - t * kKeyTile;  // 1..63
    const unsigned char* tile = kbase + (size_t)t * kKeyTile * kstride;
    __syncthreads();  // every wave is done reading both buffers
    ST::run_rows(lds0, wave, lane, [=](int row) { return tile + (size_t)min(row, nrows - 1) * kstride; }, last_chunk);
    wait_vmem();
    __syncthreads();
    if (active) {
      for (int ks = 0; ks < 2; ks++) {
        bf16x8 kf[KS];
        read_frags<HD, KS>(kf, lds, ks, l32, hi);
#pragma unroll
        for (int s = 0; s < NQ; s++) {
          f32x16 acc;
          mfma_chain<KS, FORM == kF32>(acc, kf, qf[s]);
#pragma unroll
          for (int v = 0; v < 16; v++)
            if (ks * 32 + (v >> 2) * 8 + hi * 4 + (v & 3) >= nrows) acc[v] = kMasked;
          stats_fold<FORM>(acc, st[s], c2);
        }
      }
    }
  }

  if (causal_patch && split == 0) {
    // the patch's own keys follow the context rows; the query of patch token t = r % p sees patch
    // keys 0..t (Sec. 2.3: the patch is appended after the block and attends causally)
    const int ptiles = (pl.p + kKeyTile - 1) / kKeyTile;
    for (int pt = 0; pt < ptiles; pt++) {
      const int nrows = min(kKeyTile, pl.p - pt * kKeyTile);
      const unsigned char* tile = kbase + (size_t)(N + pt * kKeyTile) * kstride;
      __syncthreads();  // every wave is done reading the buffer this tile lands in
      ST::run_rows(lds0, wave, lane, [=](int row) { return tile + (size_t)min(row, nrows - 1) * kstride; }, last_chunk);
      wait_vmem();
      __syncthreads();
      if (active) {
        for (int ks = 0; ks < 2; ks++) {
          bf16x8 kf[KS];
          read_frags<HD, KS>(kf, lds, ks, l32, hi);
#pragma unroll
          for (int s = 0; s < NQ; s++) {
            int g, t_row;
            head_and_token(pl.p, pl.inv_p, min(row0 + s * 32 + l32, pl.R - 1), g, t_row);
            f32x16 acc;
            mfma_chain<KS, FORM == kF32>(acc, kf, qf[s]);
#pragma unroll
            for (int v = 0; v < 16; v++)
              if (pt * kKeyTile + ks * 32 + (v >> 2) * 8 + hi * 4 + (v & 3) > t_row) acc[v] = kMasked;
            stats_fold<FORM>(acc, st[s], c2);
          }
        }
      }
    }
  }

  if (!active) return;
#pragma unroll
  for (int s = 0; s < NQ; s++) {
    // lanes l and l^32 hold the same query row over disjoint keys
    const float mo = __shfl_xor(st[s].m, 32), Do = __shfl_xor(st[s].D, 32);
    const float mn = fmaxf(st[s].m, mo);
    const float Dn = st[s].D * correction<FORM>(st[s].m, mn, c2) + Do * correction<FORM>(mo, mn, c2);
    const int r = row0 + s * 32 + l32;
    if (hi == 0 && r < pl.R)
      out[((size_t)bh * n_splits + split) * Rpad + r] = make_float2(mn * c2, Dn);
  }
}

// ------------------------------------------------------- between the passes
// A row's reference (in units of the exponent) and sum from its key splits, for ROWS rows at a time (r0, r0 + step, ..;
// rows beyond R repeat the last one).  AT_ONCE splits of every row are loaded together.
template <int ROWS, int AT_ONCE>
__device__ __forceinline__ void combine_splits(float (&mx)[ROWS], float (&den)[ROWS], const float2* st, int r0, int step,
                                               const Plan& pl) {
#pragma unroll
  for (int i = 0; i < ROWS; i++) mx[i] = kMasked, den[i] = 0.f;
  for (int s0 = 0; s0 < pl.live_splits; s0 += AT_ONCE) {
    float2 e[ROWS][AT_ONCE];
#pragma unroll
    for (int i = 0; i < ROWS; i++)
#pragma unroll
      for (int j = 0; j < AT_ONCE; j++)
        e[i][j] = st[(size_t)min(s0 + j, pl.live_splits - 1) * pl.Rpad + min(r0 + i * step, pl.R - 1)];
#pragma unroll
    for (int i = 0; i < ROWS; i++) {
      float m = mx[i];
#pragma unroll
      for (int j = 0; j < AT_ONCE; j++) m = fmaxf(m, e[i][j].x);
      float sum = den[i] * ex2(mx[i] - m);
#pragma unroll
      for (int j = 0; j < AT_ONCE; j++)
        sum += s0 + j < pl.live_splits ? e[i][j].y * ex2(e[i][j].x - m) : 0.f;
      mx[i] = m, den[i] = sum;
    }
  }
}

// One thread per row.  Only where pass 2 runs over several rounds of workgroups (launch_rows).  kFolded: the rows'
// log-sum-exps, rows of a head dense, to `lse`; otherwise the combined pair takes the place of the first split's.
template <int FORM>
__global__ void combine_row_stats(float2* stats, float* __restrict__ lse, Plan pl, int total) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= total) return;
  const int bh = i / pl.R, r = i - bh * pl.R;
  float2* st = stats + (size_t)bh * pl.n_splits * pl.Rpad;
  float m[1], den[1];
  combine_splits<1, 8>(m, den, st, r, 0, pl);
  if (FORM == kFolded) lse[i] = m[0] + __log2f(den[0]);
  else st[r] = make_float2(m[0], den[0]);
}

// Fills LDS with what pass 2 needs of every row, from row_lse * lse_scale (the caller's natural-log normalisers, or
// combined ones) or, if that is null, from the key splits of pass 1.  first[r] is added to every scaled logit of row r:
// minus its base-2 log-sum-exp or (other than kFolded) minus its reference, in which case second[r] is 1 / sum.  Rows
// beyond R get -inf and 0 (weight 0).  In two parts: request() asks for the first rows ahead of the workgroup's other
// loads, finish() comes behind them, so that its wait is not for those (they return in order).
template <int FORM, int THREADS, int ROWS>
struct NormFill {
  float early[ROWS];  // rows threadIdx.x + i * THREADS

  __device__ __forceinline__ void request(const float* __restrict__ row_lse, int bh, const Plan& pl) {
    if (!row_lse) return;
#pragma unroll
    for (int i = 0; i < ROWS; i++) early[i] = row_lse[(size_t)bh * pl.R + min((int)threadIdx.x + i * THREADS, pl.R - 1)];
  }
  __device__ __forceinline__ void finish(float* first, float* second, int rows, const float2* __restrict__ stats,
                                         const float* __restrict__ row_lse, float lse_scale, int bh, const Plan& pl) {
    auto put = [&](int r, float m, float inv) {
      if (r >= rows) return;
      first[r] = r < pl.R ? -m : -INFINITY;
      if (FORM != kFolded) second[r] = r < pl.R ? inv : 0.f;
    };
    if (row_lse) {
#pragma unroll
      for (int i = 0; i < ROWS; i++) put(threadIdx.x + i * THREADS, early[i] * lse_scale, 1.f);
      for (int r = threadIdx.x + ROWS * THREADS; r < rows; r += THREADS)
        put(r, row_lse[(size_t)bh * pl.R + min(r, pl.R - 1)] * lse_scale, 1.f);
      return;
    }
    auto fill = [&](auto rows_c, auto splits_c) {
      constexpr int kAtOnce = decltype(rows_c)::value, kSplits = decltype(splits_c)::value;
      for (int r0 = threadIdx.x; r0 < rows; r0 += kAtOnce * THREADS) {
        float m[kAtOnce], den[kAtOnce];
        combine_splits<kAtOnce, kSplits>(m, den, stats + (size_t)bh * pl.n_splits * pl.Rpad, r0, THREADS, pl);
#pragma unroll
        for (int i = 0; i < kAtOnce; i++) {
          if (FORM == kFolded) put(r0 + i * THREADS, m[i] + __log2f(den[i]), 0.f);
          else put(r0 + i * THREADS, m[i], 1.0f / den[i]);
        }
      }
    };
    constexpr std::integral_constant<int, 1> one;
    constexpr std::integral_constant<int, 2> two;
    constexpr std::integral_constant<int, 8> eight;
    constexpr std::integral_constant<int, 16> sixteen;
    // Where a thread has one row, more than 8 splits of it are loaded 16 at a time: every batch is a round trip that the
    // workgroup waits for (8 heads of 192 rows, 32 splits: pass 2 9.4 -> 8.5 us; with 8 splits 16 are 0.2 us longer).
    // With two rows a thread from 25 splits on, where it makes two of four batches (both passes, 8 / 16 at a time: 1 head of 512 rows,
    // 4000 keys in 32 splits 16.4 / 16.0 us, 2 heads of 288 rows, 9000 keys in 29 18.2 / 17.7; in 17 to 24 splits, three batches or two,
    // 8 heads of 288 rows, 9000 keys 27.7 / 29.2, 1 head, 2500 keys 14.3 / 14.6).
    if constexpr (ROWS > 1) {
      if (pl.live_splits > 24 && pl.R <= 2 * THREADS) fill(two, sixteen);
      else fill(two, eight);
    } else if (pl.live_splits > 8) fill(one, sixteen);
    else fill(one, eight);
  }
};

// ------------------------------------------------------------------ pass 2
// What pass 2 knows of the 16 query rows that a lane holds of an accumulator tile (NormFill).
template <int FORM>
struct RowNorms {
  float first[16], second[FORM == kFolded ? 1 : 16];
};

// Column reduction of the previous accumulator tile (16 query rows of one key), sliced like the statistics above.
// kFolded takes the maximum over the exponents, the other forms over the weights.
template <int FORM, int REDUCE>
struct Column {
  static constexpr bool kMax = REDUCE == EPICACHE_REDUCE_MAX, kLog = kMax && FORM == kFolded;
  static constexpr float kNeutral = kLog ? -INFINITY : 0.f;
  __device__ static __forceinline__ float merge(float a, float b) { return kMax ? fmaxf(a, b) : a + b; }
  __device__ static __forceinline__ float score(float x) { return kLog ? ex2(x) : x; }
};

template <int FORM, int REDUCE>
__device__ __forceinline__ float col_group(const f32x16& P, const RowNorms<FORM>& nl, int g, float c2) {
  using C = Column<FORM, REDUCE>;
  float x[4];
#pragma unroll
  for (int i = 0; i < 4; i++) {
    x[i] = fmaf(P[4 * g + i], c2, nl.first[4 * g + i]);
    if (!C::kLog) x[i] = ex2(x[i]);
    if (FORM != kFolded) x[i] *= nl.second[FORM != kFolded ? 4 * g + i : 0];
  }
  if (C::kMax) return vmax(vmax3(x[0], x[1], x[2]), x[3]);
  return (x[0] + x[1]) + (x[2] + x[3]);
}

template <int FORM, int REDUCE>
__device__ __forceinline__ void col_fold(const f32x16& P, const RowNorms<FORM>& nl, float& col, float c2) {
  const float a = col_group<FORM, REDUCE>(P, nl, 0, c2), b = col_group<FORM, REDUCE>(P, nl, 1, c2);
  const float c = col_group<FORM, REDUCE>(P, nl, 2, c2), d = col_group<FORM, REDUCE>(P, nl, 3, c2);
  if (REDUCE == EPICACHE_REDUCE_MAX) col = vmax3(vmax3(a, b, c), d, col);
  else col = col + ((a + b) + (c + d));
}

template <int LO, int HI>
__device__ __forceinline__ void col_stage_fma(float (&x)[16], const f32x16& P, const float (&nl)[16], float c2) {
#pragma unroll
  for (int v = LO; v < HI; v++) x[v] = fmaf(P[v], c2, nl[v]);
#pragma unroll
  for (int v = LO; v < HI; v++) pin(x[v]);
}

// weights into the column: the exponentials as they are (kFolded) or times the rows' 1 / sum
template <int FORM, int REDUCE, int LO, int HI>
__device__ __forceinline__ void col_stage_add(float (&x)[16], const RowNorms<FORM>& nl, float& s0, float& s1) {
  if constexpr (FORM == kFolded) {
    stage_add<LO, HI>(x, s0, s1);
  } else if constexpr (REDUCE == EPICACHE_REDUCE_MAX) {
#pragma unroll
    for (int v = LO; v < HI; v++) x[v] *= nl.second[v];
#pragma unroll
    for (int v = LO; v < HI; v++) pin(x[v]);
    stage_max<LO, HI>(x, s0, s1);
  } else {
#pragma unroll
    for (int v = LO; v < HI; v++) {
      float& s = v & 1 ? s1 : s0;
      s = fmaf(x[v], nl.second[v], s);
    }
    if (HI > LO) pin(s0), pin(s1);
  }
}

template <int FORM, int KS, int REDUCE, int J>
__device__ __forceinline__ void reduce_slot(f32x16& acc, const bf16x8 (&a)[KS], const bf16x8 (&b)[KS],
                                            const f32x16& P, const RowNorms<FORM>& nl, float c2, float (&x)[16],
                                            float& s0, float& s1) {
  using SL = Slots<KS>;
  if (J == 0) acc = f32x16{0};
  mfma_step<FORM == kF32>(acc, a[J], b[J]);
  fence_sched();
  col_stage_fma<SL::reduce(J), SL::reduce(J + 1)>(x, P, nl.first, c2);
  if constexpr (Column<FORM, REDUCE>::kLog) {
    if constexpr (J >= 1) stage_max<SL::reduce(J - 1), SL::reduce(J)>(x, s0, s1);
  } else {
    if constexpr (J >= 1) stage_exp<SL::reduce(J - 1), SL::reduce(J)>(x);
    if constexpr (J >= 2) col_stage_add<FORM, REDUCE, SL::reduce(J - 2), SL::reduce(J - 1)>(x, nl, s0, s1);
  }
  fence_sched();
}

// `late` runs behind the first quarter of the MFMAs
template <int FORM, int KS, int REDUCE, int J = 0, typename Late>
__device__ __forceinline__ void reduce_slots(f32x16& acc, const bf16x8 (&a)[KS], const bf16x8 (&b)[KS],
                                             const f32x16& P, const RowNorms<FORM>& nl, float c2, float (&x)[16],
                                             float& s0, float& s1, Late late) {
  if constexpr (J == KS / 4) late();
  reduce_slot<FORM, KS, REDUCE, J>(acc, a, b, P, nl, c2, x, s0, s1);
  if constexpr (J + 1 < KS) reduce_slots<FORM, KS, REDUCE, J + 1>(acc, a, b, P, nl, c2, x, s0, s1, late);
}

struct Nothing {
  __device__ __forceinline__ void operator()() const {}
};

// acc <- MFMA chain, interleaved with reducing P (the tile finished one unit earlier; nl: what its 16 rows are
// normalised with) into `col`.
template <int FORM, int KS, int REDUCE, typename Late = Nothing>
__device__ __forceinline__ void reduce_unit(f32x16& acc, const bf16x8 (&a)[KS], const bf16x8 (&b)[KS],
                                            const f32x16& P, const RowNorms<FORM>& nl, float& col, float c2,
                                            Late late = Late{}) {
  using SL = Slots<KS>;
  using C = Column<FORM, REDUCE>;
  float x[16];
  float s0 = C::kNeutral, s1 = s0;
  reduce_slots<FORM, KS, REDUCE>(acc, a, b, P, nl, c2, x, s0, s1, late);
  if constexpr (C::kLog) {
    stage_max<SL::reduce(KS - 1), SL::reduce(KS)>(x, s0, s1);
  } else {
    stage_exp<SL::reduce(KS - 1), SL::reduce(KS)>(x);
    col_stage_add<FORM, REDUCE, SL::reduce(KS - 2), SL::reduce(KS - 1)>(x, nl, s0, s1);
    col_stage_add<FORM, REDUCE, SL::reduce(KS - 1), SL::reduce(KS)>(x, nl, s0, s1);
  }
  if constexpr (C::kMax) col = vmax3(col, s0, s1);
  else col += s0 + s1;
  fence_sched();
}

// quarters G0 .. G1 - 1 of what a lane holds
template <int G0 = 0, int G1 = 4>
__device__ __forceinline__ void read_rows(float (&x)[16], const float* rows, int row0, int hi) {
#pragma unroll
  for (int g4 = G0; g4 < G1; g4++) {
    const float4 v = *reinterpret_cast<const float4*>(rows + row0 + g4 * 8 + hi * 4);
    x[g4 * 4 + 0] = v.x, x[g4 * 4 + 1] = v.y, x[g4 * 4 + 2] = v.z, x[g4 * 4 + 3] = v.w;
  }
}
// Query tiles in LDS at a time.  With two numbers per row the 12288 rows and more of a call leave room for one tile of
// 512-byte rows only (160 KB: 2 x 32 KB and 8 bytes a row).
template <int FORM> constexpr __host__ __device__ int norms_per_row() { return FORM == kFolded ? 1 : 2; }
template <int FORM, int HD>
__host__ __device__ __forceinline__ int query_tiles(const Plan& pl) {
  return FORM != kFolded && HD == 256 && pl.Rpad > 12288 ? 1 : 2;
}
// the second numbers of all `rows` rows follow the first ones
template <int FORM>
__device__ __forceinline__ void read_norms(RowNorms<FORM>& nl, const float* first, int rows, int row0, int hi) {
  read_rows(nl.first, first, row0, hi);
  if constexpr (FORM != kFolded) read_rows(nl.second, first + rows, row0, hi);
}

// NK 32-key sub-tiles per wave (1 for rows of more than 128 elements: the registers), 4 waves in RG groups.  A group takes every
// RG-th query tile, through LDS tiles of its own, and its 4 / RG waves have keys of their own: with few keys in the call (few
// heads, or short ones) more workgroups with shorter ways (row_groups in launch_rules.h).
template <int FORM, int HD, int KS, int NK, int REDUCE, int RG>
__global__ __launch_bounds__(256, 2) void score_reduce(const bf16_t* __restrict__ q,
                                                       const bf16_t* __restrict__ k,
                                                       const float2* __restrict__ stats,
                                                       const float* __restrict__ row_lse, float lse_scale,
                                                       float* __restrict__ scores, Plan pl) {
  using TL = Tile<HD>;
  using C = Column<FORM, REDUCE>;
  constexpr int kWaves = 4 / RG;           // of a group
  constexpr int kKeys = 32 * NK * kWaves;  // keys per workgroup
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  unsigned char* lds = smem;                                            // query tiles, then what NormFill makes:
  float* norms = reinterpret_cast<float*>(smem + RG * query_tiles<FORM, HD>(pl) * TL::kTileBytes);  // [Rpad] or [2][Rpad]
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave_of_all = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int group = wave_of_all / kWaves, wave = wave_of_all % kWaves;
  const int l32 = lane & 31, hi = lane >> 5;
  // XCD-aware ids as in pass 1: the key blocks of one (b, h) all stream the same query rows through LDS
  // and are given ids that land on one XCD: id = xcd + 8 * (key block + NKB * (bh / 8)), bh % 8 = xcd.
  int kb = blockIdx.x >> 3, bh = blockIdx.y * 8 + (blockIdx.x & 7);
  if (pl.spread) spread_parts(blockIdx.x, (pl.N + kKeys - 1) / kKeys, bh, kb);
  if (bh >= pl.nb * pl.Hkv) return;
  const int b = batch_of(pl, bh), h = bh - b * pl.Hkv;
  const int N = ctx_rows(pl, bh);
  clear_claims(pl, bh, kb == 0);  // also of a head without keys
  if (kb * kKeys >= N) return;    // a shorter head of a ragged batch: no keys here
  const int key0 = kb * kKeys + wave * (32 * NK);
  const float c2 = pl.c2;

  using ST = Stager<HD, KS, kWaves, FORM == kFolded>;
  const unsigned char* qbase = reinterpret_cast<const unsigned char*>(q + b * pl.qsb + (int64_t)(h * pl.G) * pl.qsh);
  const size_t qsh = (size_t)pl.qsh * 2;
  const uint32_t qstride = (uint32_t)pl.qst * 2;
  const int p = pl.p, last_row = pl.R - 1;
  // In registers before the loop: a scalar load inside it or right in front of it shares its counter with the LDS
  // reads, which could then only be waited for all at once.  (As the code stands no time shows either way: pass 2 of 128
  // heads, R = 512, N = 8192 139 us.)
  float inv_p = pl.inv_p;
  float* out = scores + (size_t)bh * pl.N;
  asm volatile("" : "+s"(inv_p), "+s"(out));
  const bool dense_tiles = p % 64 == 0;  // every 64-row tile lies inside one query head
  const int last_chunk = pl.d / 8 - 1;
  const typename ST::Offsets qoff = ST::offsets(wave, lane, qstride, last_chunk);
  lds += group * 2 * TL::kTileBytes;
  const uint32_t lds0 = lds_address(smem) + group * 2 * TL::kTileBytes;
  // dense tiles are staged in order (RG = 1), so the address of the next one is carried along instead of being derived
  // from the tile index with a division per tile
  const unsigned char* qtile = qbase;  // first row of the next tile to stage
  int qtile_row = 0;                   // that row's index within its query head
  auto stage_queries = [&](uint32_t dst, int t) {
    if (RG > 1 && dense_tiles) {
      int g, tok;
      head_and_token(p, inv_p, t * 64, g, tok);
      g = __builtin_amdgcn_readfirstlane(g), tok = __builtin_amdgcn_readfirstlane(tok);
      ST::run(dst, qbase + (size_t)g * qsh + (size_t)tok * qstride, qoff, wave);
    } else if (dense_tiles) {
      ST::run(dst, qtile, qoff, wave);
      qtile_row += 64;
      if (qtile_row == p) {
        qtile_row = 0;
        qtile += qsh - (size_t)(p - 64) * qstride;  // first row of the next query head
      } else {
        qtile += (size_t)64 * qstride;
      }
    } else {
      // rows beyond R re-read the last row; their -lse is -inf, so they contribute nothing
      ST::run_rows(dst, wave, lane, [=](int row) {
        int g, tok;
        head_and_token(p, inv_p, min(t * 64 + row, last_row), g, tok);
        return qbase + (size_t)g * qsh + (size_t)tok * qstride;
      }, last_chunk);
    }
  };
  const int qtiles = pl.Rpad / 64;
  if (RG == 1 || group < qtiles) stage_queries(lds0, group);

  NormFill<FORM, 256, 5> fill;
  fill.request(row_lse, bh, pl);

  // key fragments of this wave stay in registers for the whole query loop
  const bf16_t* kbase = k + b * pl.ksb + (int64_t)h * pl.ksh;
  bf16x8 kf[NK][KS];
#pragma unroll
  for (int s = 0; s < NK; s++)
    load_row_frags<KS>(kf[s], kbase + (int64_t)min(key0 + s * 32 + l32, N - 1) * pl.kst, hi, pl.d);

  fill.finish(norms, norms + pl.Rpad, pl.Rpad, stats, row_lse, lse_scale, bh, pl);

  // The fragments are used here, i.e. loaded before the wait below.  Left to itself the compiler sinks these
  // loads behind the barrier, finds them outstanding at the loop's entry and puts a counted wait in front of the
  // first use of each inside the loop; from the second iteration on those waits only see the tile in flight and
  // make every wave wait for it a unit and a half after it was requested.
#pragma unroll
  for (int s = 0; s < NK; s++)
#pragma unroll
    for (int j = 0; j < KS; j++) asm volatile("" : "+v"(kf[s][j]));

  // running sum or maximum of weights, or (kFolded) maximum of the base-2 log weights: exp2 is monotone, so one
  // exponential per key at the end is enough
  float col[NK];
#pragma unroll
  for (int s = 0; s < NK; s++) col[s] = C::kNeutral;
  f32x16 accA, accB;
#pragma unroll
  for (int v = 0; v < 16; v++) accA[v] = accB[v] = 0.f;
  // nlP: of the last unit's rows, nlC: of the rows before those.  The "tile before the first" has weight 0.
  RowNorms<FORM> nlP, nlC;
#pragma unroll
  for (int v = 0; v < 16; v++) {
    nlP.first[v] = -INFINITY;
    if (FORM != kFolded) nlP.second[v] = 0.f;
  }

  wait_vmem();
  __syncthreads();  // query tile 0 and norms[] are in LDS

  int buf = 0;
  // Units of one query tile: (qs, s) for qs in {0,1} (32-row halves), s in {0,1} (key halves of the
  // wave): u = 2*qs + s accumulates into accA (u even) / accB (u odd) while unit u-1 is reduced.
  for (int t = group; t - group < qtiles; t += RG) {
    const unsigned char* cur = lds + buf * TL::kTileBytes;
    const bool two = query_tiles<FORM, HD>(pl) == 2;
    if (two && t + RG < qtiles) stage_queries(lds0 + (buf ^ 1) * TL::kTileBytes, t + RG);
    if (RG > 1 && t >= qtiles) {  // none left for this group
    } else if constexpr (NK == 2 && FORM == kFolded) {
      bf16x8 qf0[KS], qf1[KS];
      read_frags<HD, KS>(qf0, cur, 0, l32, hi);
      read_frags<HD, KS>(qf1, cur, 1, l32, hi);
      read_norms<FORM>(nlC, norms, pl.Rpad, t * 64, hi);
      // unit 0: rows qs=0, keys s=0; previous unit = (prev tile, qs=1, s=1) with nlP
      reduce_unit<FORM, KS, REDUCE>(accA, qf0, kf[0], accB, nlP, col[1], c2);
      read_norms<FORM>(nlP, norms, pl.Rpad, t * 64 + 32, hi);
      reduce_unit<FORM, KS, REDUCE>(accB, qf0, kf[1], accA, nlC, col[0], c2);
      reduce_unit<FORM, KS, REDUCE>(accA, qf1, kf[0], accB, nlC, col[1], c2);
      reduce_unit<FORM, KS, REDUCE>(accB, qf1, kf[1], accA, nlP, col[0], c2);
    } else if constexpr (NK == 2) {  // two numbers per row: one set of them and one query half in registers at a time
      bf16x8 qf[KS];
      read_frags<HD, KS>(qf, cur, 0, l32, hi);
      reduce_unit<FORM, KS, REDUCE>(accA, qf, kf[0], accB, nlP, col[1], c2);
      read_norms<FORM>(nlP, norms, pl.Rpad, t * 64, hi);
      reduce_unit<FORM, KS, REDUCE>(accB, qf, kf[1], accA, nlP, col[0], c2);
      read_frags<HD, KS>(qf, cur, 1, l32, hi);
      reduce_unit<FORM, KS, REDUCE>(accA, qf, kf[0], accB, nlP, col[1], c2);
      read_norms<FORM>(nlP, norms, pl.Rpad, t * 64 + 32, hi);
      reduce_unit<FORM, KS, REDUCE>(accB, qf, kf[1], accA, nlP, col[0], c2);
    } else {
      bf16x8 qf[KS];
      read_frags<HD, KS>(qf, cur, 0, l32, hi);
      reduce_unit<FORM, KS, REDUCE>(accA, qf, kf[0], accB, nlP, col[0], c2);
      read_norms<FORM>(nlP, norms, pl.Rpad, t * 64, hi);
      read_frags<HD, KS>(qf, cur, 1, l32, hi);
      reduce_unit<FORM, KS, REDUCE>(accB, qf, kf[0], accA, nlP, col[0], c2);
      read_norms<FORM>(nlP, norms, pl.Rpad, t * 64 + 32, hi);
    }
    if (!two && t + 1 < qtiles) {
      __syncthreads();  // the one tile has been read by every wave
      stage_queries(lds0, t + 1);
    }
    wait_vmem();
    __syncthreads();
    if (two) buf ^= 1;
  }
  col_fold<FORM, REDUCE>(accB, nlP, col[NK - 1], c2);  // last unit (qs=1, s=1)

  if constexpr (RG > 1) {
    float* part = reinterpret_cast<float*>(smem);  // [RG][kKeys]; the tiles have been read
#pragma unroll
    for (int s = 0; s < NK; s++) {
      const float o = __shfl_xor(col[s], 32);
      if (hi == 0) part[group * kKeys + wave * (32 * NK) + s * 32 + l32] = C::merge(col[s], o);
    }
    __syncthreads();
    const int key = kb * kKeys + tid;
    if (tid < kKeys && key < N) {
      float x = part[tid];
#pragma unroll
      for (int g = 1; g < RG; g++) x = C::merge(x, part[g * kKeys + tid]);
      out[key] = C::score(x);
    }
    return;
  }
#pragma unroll
  for (int s = 0; s < NK; s++) {
    // lanes l and l^32 hold the same key over disjoint query rows
    const float o = __shfl_xor(col[s], 32);
    const int key = key0 + s * 32 + l32;
    if (hi == 0 && key < N) out[key] = C::score(C::merge(col[s], o));
  }
}

// ------------------------------------------------------- pass 2, streaming form
// For R <= 256 (all query rows of a KV head fit one workgroup): same data flow as pass 1 - query
// fragments stay in registers, 64-key tiles stream through LDS - with the operands swapped so that
// a lane owns one key column and 16 query rows.  Each wave reduces its own rows; the per-key
// partial results of the NW waves meet in LDS once per tile.  Reads K with fully coalesced
// 1 KiB bursts, which the key-stationary form above cannot do when R is small.
template <int FORM, int HD, int KS, int NQ, int NW, int REDUCE>
__global__ __launch_bounds__(NW * 64, (NW == 1 || (HD > 128 && NW < 4) ? 1 : 2)) void score_reduce_stream(const bf16_t* __restrict__ q,
                                                                  const bf16_t* __restrict__ k,
                                                                  const float2* __restrict__ stats,
                                                                  const float* __restrict__ row_lse, float lse_scale,
                                                                  float* __restrict__ scores, Plan pl) {
  using TL = Tile<HD>;
  using ST = Stager<HD, KS, NW, FORM == kFolded>;
  constexpr int kRows = 32 * NQ * NW;
  using C = Column<FORM, REDUCE>;
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  unsigned char* lds = smem;                                             // 2 key tiles
  float* norms = reinterpret_cast<float*>(smem + 2 * TL::kTileBytes);    // [kRows] or [2][kRows]
  float(*part)[NW][64] = reinterpret_cast<float(*)[NW][64]>(norms + norms_per_row<FORM>() * kRows);  // [2]
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, hi = lane >> 5;
  int split = blockIdx.x >> 3, bh = blockIdx.y * 8 + (blockIdx.x & 7);  // a head's splits on one XCD, as above
  if (pl.spread) spread_parts(blockIdx.x, pl.reduce_splits, bh, split);
  if (bh >= pl.nb * pl.Hkv) return;
  const int b = batch_of(pl, bh), h = bh - b * pl.Hkv;
  const int row0 = wave * (32 * NQ);
  const bool active = row0 < pl.R;
  const float c2 = pl.c2;

  const int N = ctx_rows(pl, bh);
  const int tiles = (N + kKeyTile - 1) / kKeyTile;
  const int tiles_per_split = split_length(pl, tiles, pl.reduce_splits, pl.reduce_tiles_per_split);
  const int t_begin = split * tiles_per_split;
  const int t_end = min(tiles, t_begin + tiles_per_split);
  clear_claims(pl, bh, split == 0);  // also of a head without keys
  if (t_begin >= t_end) return;      // a shorter head of a ragged batch: no keys in this split

  const unsigned char* kbase = reinterpret_cast<const unsigned char*>(k + b * pl.ksb + (int64_t)h * pl.ksh);
  const uint32_t kstride = (uint32_t)pl.kst * 2;
  const int last_chunk = pl.d / 8 - 1;
  const typename ST::Offsets koff = ST::offsets(wave, lane, kstride, last_chunk);
  const uint32_t lds0 = lds_address(lds);
  auto stage_keys = [&](uint32_t dst, int t) {
    const unsigned char* tile = kbase + (size_t)t * kKeyTile * kstride;
    const int nrows = N - t * kKeyTile;
    if (nrows >= kKeyTile) ST::run(dst, tile, koff, wave);
    else  // ragged last tile: rows beyond N re-read the last key; their results are never written
      ST::run_rows(dst, wave, lane, [=](int row) { return tile + (size_t)min(row, nrows - 1) * kstride; }, last_chunk);
  };
  stage_keys(lds0, t_begin);

  NormFill<FORM, NW * 64, (kRows + NW * 64 - 1) / (NW * 64)> fill;
  fill.request(row_lse, bh, pl);

  // query fragments (A operand: rows = queries) stay in registers for the whole key loop; rows beyond R have weight 0
  bf16x8 qf[NQ][KS];
#pragma unroll
  for (int s = 0; s < NQ; s++) {
    int g, t;
    head_and_token(pl.p, pl.inv_p, min(row0 + s * 32 + l32, pl.R - 1), g, t);
    load_row_frags<KS>(qf[s], q + b * pl.qsb + (int64_t)(h * pl.G + g) * pl.qsh + (int64_t)t * pl.qst, hi, pl.d);
  }

  fill.finish(norms, norms + kRows, kRows, stats, row_lse, lse_scale, bh, pl);

  wait_vmem();
  __syncthreads();  // first key tile and norms[] are in LDS

  // The pipeline runs across tile boundaries: the last unit of tile t-1 (in accB) is reduced while the first
  // chain of tile t is issued, so the column partials of a tile are complete one unit into the next tile and
  // its scores are written one barrier later than its keys were consumed.
  auto exchange = [&](const float (&c)[2], int t) {  // this wave's partials of tile t -> part[t & 1]
#pragma unroll
    for (int ks = 0; ks < 2; ks++) {
      // lanes l and l^32 hold the same key over disjoint query rows; the swap leaves the lower half's values
      // in both halves of one register and the upper half's in both halves of the other (vector ALU, no LDS)
      const unsigned int bits = __float_as_uint(c[ks]);
      const auto r = __builtin_amdgcn_permlane32_swap(bits, bits, false, false);
      const float lo = __uint_as_float(r[0]), up = __uint_as_float(r[1]);
      if (hi == 0) part[t & 1][wave][ks * 32 + l32] = C::merge(lo, up);
    }
  };
  auto write_scores = [&](int t) {  // after the barrier that completes part[t & 1]
    if (tid < 64) {
      const int key = t * kKeyTile + tid;
      if (key < N) {
        float v = part[t & 1][0][tid];
#pragma unroll
        for (int w = 1; w < NW; w++)
          v = C::merge(v, part[t & 1][w][tid]);
        scores[(size_t)bh * pl.N + key] = C::score(v);
      }
    }
  };

  int buf = 0;
  f32x16 accA, accB;                             // accB after a tile: its last unit, still to be reduced
#pragma unroll
  for (int v = 0; v < 16; v++) accB[v] = kMasked;  // before the first tile: a filler whose weights are 0; what it
                                                   // leaves in cs_prev is never exchanged
  float cs_prev[2] = {C::kNeutral, C::kNeutral};  // partials of the previous tile (keys ks*32 + l32)
  for (int t = t_begin; t < t_end; t++) {
    const unsigned char* cur = lds + buf * TL::kTileBytes;
    if (t + 1 < t_end) stage_keys(lds0 + (buf ^ 1) * TL::kTileBytes, t + 1);
    float cs[2] = {C::kNeutral, C::kNeutral};  // this wave's rows, keys ks*32 + l32 of the tile
    if (active) {
      // units (ks, s): key half ks, query sub-tile s; unit u accumulates into accA/accB (u even/odd)
      // while unit u-1 is reduced over its 16 rows into cs[ks of u-1]
      // Two numbers per row and rows of 512 bytes exceed the registers by a few: the last quarter of the fragments
      // takes the first one's place as its MFMAs have been issued (both passes over 32 heads, R = 128, N = 4096,
      // d = 256: 47 -> 29 us), and half of the second numbers come with it.
      constexpr bool kLate = FORM != kFolded && KS == 16 && NQ == 1;
      constexpr int kNow = kLate ? KS * 3 / 4 : KS;
      bf16x8 kf[KS];
      read_frags<HD, KS, 0, kNow>(kf, cur, 0, l32, hi);
#pragma unroll
      for (int u = 0; u < 2 * NQ; u++) {
        const int s = u % NQ, sp = (u + 2 * NQ - 1) % NQ, ksp = (u - 1) / NQ;
        if (u == NQ) read_frags<HD, KS, 0, kNow>(kf, cur, 1, l32, hi);
        RowNorms<FORM> nl;  // of the 16 rows this lane holds of the previous unit
        read_rows(nl.first, norms, row0 + sp * 32, hi);
        if constexpr (FORM != kFolded) read_rows<0, kLate ? 2 : 4>(nl.second, norms + kRows, row0 + sp * 32, hi);
        auto late = [&] {
          if constexpr (!kLate) return;
          else {
            read_frags<HD, KS, kNow, KS>(kf, cur, u / NQ, l32, hi);
            read_rows<2, 4>(nl.second, norms + kRows, row0 + sp * 32, hi);
          }
        };
        if (u == 0) {
          reduce_unit<FORM, KS, REDUCE>(accA, qf[0], kf, accB, nl, cs_prev[1], c2, late);  // last unit of tile t-1
        } else if (u & 1) {
          reduce_unit<FORM, KS, REDUCE>(accB, qf[s], kf, accA, nl, cs[ksp], c2, late);
        } else {
          reduce_unit<FORM, KS, REDUCE>(accA, qf[s], kf, accB, nl, cs[ksp], c2, late);
        }
      }
    }
    if (t > t_begin) exchange(cs_prev, t - 1);
    wait_vmem();
    __syncthreads();  // tile t+1 staged, part[(t-1) & 1] complete; it is rewritten two barriers from now
    if (t > t_begin) write_scores(t - 1);
    cs_prev[0] = cs[0], cs_prev[1] = cs[1];
    buf ^= 1;
  }
  if (active) {
    RowNorms<FORM> nl;
    read_norms<FORM>(nl, norms, kRows, row0 + (NQ - 1) * 32, hi);
    col_fold<FORM, REDUCE>(accB, nl, cs_prev[1], c2);  // last unit of the last tile: odd index, key half 1
  }
  exchange(cs_prev, t_end - 1);
  __syncthreads();
  write_scores(t_end - 1);
}

// The key splits become one number per row in every workgroup of pass 2 while its keys are on their way, or, where the
// chip takes more than one round of those workgroups, in a kernel of its own between the passes: 5 us and a launch, against
// 2 us per round (64 heads of 512 rows, 8192 keys, 4 rounds: pass 2 80 -> 89 us).  The streaming form always has one round
// (32 heads of 192 rows, 4096 keys: 8.0 + 14.8 us with the kernel in between, 14.9 us without).  nk: 32-key groups per wave.
bool streams_keys(const Plan& pl) { return pl.R <= pl.stats_rows_per_wg; }
int64_t blocks_of_keys(const Plan& pl, int nk) { return (pl.N + 128 * nk - 1) / (128 * nk); }
bool combines_between(const Plan& pl, bool with_lse, int nk) {
  return !with_lse && !streams_keys(pl) && blocks_of_keys(pl, nk) * pl.nb * pl.Hkv > 2 * 256;
}
// The rows' combined log-sum-exps, behind the splits' records.
float* combined_lse(const Plan& pl, float2* stats) {
  return reinterpret_cast<float*>(stats + (size_t)pl.nb * pl.Hkv * pl.n_splits * pl.Rpad);
}

// Launches with more dynamic LDS than the default limit of 64 KB raise it first.
template <typename Kernel, typename... Args>
hipError_t launch_lds(Kernel kernel, dim3 grid, int threads, size_t smem, hipStream_t stream, Args... args) {
  if (smem > 64 * 1024) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)smem);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(kernel, grid, dim3(threads), smem, stream, args...);
  return hipGetLastError();
}

template <int FORM, int HD, int KS, int NQ, int NW>
hipError_t launch_rows(const Plan& pl, const bf16_t* q, const bf16_t* k, float* scores, float2* stats,
                       const float* row_lse, hipStream_t stream) {
  using TL = Tile<HD>;
  const int bh8 = (pl.nb * pl.Hkv + 7) / 8;  // ids whose bh falls beyond the batch exit at once
  auto parts_grid = [&](int parts) { return pl.spread ? dim3(pl.nb * pl.Hkv * parts) : dim3(8 * parts, bh8); };
  if (!row_lse) {
    const int n_rb = (pl.R + 32 * NQ * NW - 1) / (32 * NQ * NW);
    const dim3 grid = pl.spread ? dim3(8 * n_rb, (pl.nb * pl.Hkv * pl.n_splits + 7) / 8) : dim3(8 * n_rb, pl.n_splits, bh8);
    hipLaunchKernelGGL((score_stats<FORM, HD, KS, NQ, NW>), grid, dim3(NW * 64), 0, stream, q, k, stats, pl);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  float lse_scale = 1.44269504088896340736f;
  Plan p2 = pl;  // pass 2
  p2.live_splits = pl.n_splits;
  if (streams_keys(pl)) {
    const dim3 grid = parts_grid(pl.reduce_splits);
    const size_t smem = 2 * TL::kTileBytes + (norms_per_row<FORM>() * 32 * NQ * NW + 2 * NW * 64) * sizeof(float);
    if (pl.reduce == EPICACHE_REDUCE_MAX)
      return launch_lds(score_reduce_stream<FORM, HD, KS, NQ, NW, EPICACHE_REDUCE_MAX>, grid, NW * 64, smem, stream, q, k,
                        stats, row_lse, lse_scale, scores, p2);
    return launch_lds(score_reduce_stream<FORM, HD, KS, NQ, NW, EPICACHE_REDUCE_SUM>, grid, NW * 64, smem, stream, q, k, stats,
                      row_lse, lse_scale, scores, p2);
  }
  constexpr int NK = HD > 128 ? 1 : 2;
  if (combines_between(pl, row_lse != nullptr, NK)) {
    float* lse = combined_lse(pl, stats);
    const int total = pl.nb * pl.Hkv * pl.R;
    hipLaunchKernelGGL(combine_row_stats<FORM>, dim3((total + 255) / 256), dim3(256), 0, stream, stats, lse, p2, total);
    if (FORM == kFolded) row_lse = lse, lse_scale = 1.0f;
    else p2.live_splits = 1;
  }
  auto launch = [&](auto groups) {
    constexpr int RG = decltype(groups)::value, kKeys = 128 * NK / RG;
    const dim3 grid = parts_grid((pl.N + kKeys - 1) / kKeys);
    const size_t smem =
        RG * query_tiles<FORM, HD>(pl) * TL::kTileBytes + (size_t)norms_per_row<FORM>() * pl.Rpad * sizeof(float);
    if (pl.reduce == EPICACHE_REDUCE_MAX)
      return launch_lds(score_reduce<FORM, HD, KS, NK, EPICACHE_REDUCE_MAX, RG>, grid, 256, smem, stream, q, k, stats, row_lse,
                        lse_scale, scores, p2);
    return launch_lds(score_reduce<FORM, HD, KS, NK, EPICACHE_REDUCE_SUM, RG>, grid, 256, smem, stream, q, k, stats, row_lse,
                      lse_scale, scores, p2);
  };
  if constexpr (FORM == kFolded) {
    switch (row_groups(pl)) {
      case 4: return launch(std::integral_constant<int, 4>{});
      case 2: return launch(std::integral_constant<int, 2>{});
    }
  }
  return launch(std::integral_constant<int, 1>{});
}

// Rows per workgroup of pass 1 (and of pass 2's streaming form) as make_plan chose them.
template <int FORM, int HD, int KS>
hipError_t launch_hd(const Plan& pl, const bf16_t* q, const bf16_t* k, float* scores, float2* stats,
                     const float* row_lse, hipStream_t stream) {
  if constexpr (HD <= 128 && FORM != kF32) {
    switch (pl.stats_rows_per_wg) {
      case 256: return launch_rows<FORM, HD, KS, 2, 4>(pl, q, k, scores, stats, row_lse, stream);
      case 192: return launch_rows<FORM, HD, KS, 3, 2>(pl, q, k, scores, stats, row_lse, stream);
    }
  }
  switch (pl.stats_rows_per_wg) {
    case 128: return launch_rows<FORM, HD, KS, 1, 4>(pl, q, k, scores, stats, row_lse, stream);
    case 64: return launch_rows<FORM, HD, KS, 1, 2>(pl, q, k, scores, stats, row_lse, stream);
    default: return launch_rows<FORM, HD, KS, 1, 1>(pl, q, k, scores, stats, row_lse, stream);
  }
}

// Row layout in LDS and 32-byte steps of the contraction; row lengths in between are padded with zeros.
template <int FORM>
hipError_t launch_rows_of(const Plan& pl, const bf16_t* q, const bf16_t* k, float* scores, float2* stats,
                          const float* row_lse, hipStream_t stream) {
  if (pl.d <= 32) return launch_hd<FORM, 64, 2>(pl, q, k, scores, stats, row_lse, stream);
  if (pl.d <= 64) return launch_hd<FORM, 64, 4>(pl, q, k, scores, stats, row_lse, stream);
  if (pl.d <= 96) return launch_hd<FORM, 128, 6>(pl, q, k, scores, stats, row_lse, stream);
  if (pl.d <= 128) return launch_hd<FORM, 128, 8>(pl, q, k, scores, stats, row_lse, stream);
  if (pl.d <= 192) return launch_hd<FORM, 256, 12>(pl, q, k, scores, stats, row_lse, stream);
  return launch_hd<FORM, 256, 16>(pl, q, k, scores, stats, row_lse, stream);
}

}  // namespace

// The place of the combined log-sum-exps (256 bytes or more a head) is free unless there are any; pass 2 then reads those
// and none of the splits' records (512 bytes or more a head).
uint32_t* claims_in_stats(const Plan& pl, float2* stats, bool with_lse) {
  static_assert(kClaimsPerHead * sizeof(uint32_t) <= 64 * sizeof(float), "Rpad is at least 64");
  const bool folded = pl.dtype == EPICACHE_DTYPE_BF16 && (pl.d == 64 || pl.d == 128);
  const bool lse_used = folded && combines_between(pl, with_lse, 2);
  return reinterpret_cast<uint32_t*>(lse_used ? static_cast<void*>(stats) : combined_lse(pl, stats));
}

hipError_t launch_score_mfma(const Plan& pl, const void* q, const void* k, float* scores, float2* stats,
                             const float* row_lse, hipStream_t stream) {
  const bf16_t* qq = static_cast<const bf16_t*>(q);
  const bf16_t* kk = static_cast<const bf16_t*>(k);
  if (pl.dtype == EPICACHE_DTYPE_BF16) {
    if (pl.d == 64) return launch_hd<kFolded, 64, 4>(pl, qq, kk, scores, stats, row_lse, stream);
    if (pl.d == 128) return launch_hd<kFolded, 128, 8>(pl, qq, kk, scores, stats, row_lse, stream);
    return launch_rows_of<kBf16>(pl, qq, kk, scores, stats, row_lse, stream);
  }
  // fp32 rows are moved as rows of twice as many two-byte units
  Plan p2 = pl;
  p2.d *= 2;
  for (int64_t* s : {&p2.qsb, &p2.qsh, &p2.qst, &p2.ksb, &p2.ksh, &p2.kst}) *s *= 2;
  return launch_rows_of<kF32>(p2, qq, kk, scores, stats, row_lse, stream);
}

}  // namespace epicache

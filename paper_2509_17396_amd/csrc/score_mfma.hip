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
#include "epicache_internal.h"
#include "mfma_tiles.h"

namespace epicache {
namespace {

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

__device__ __forceinline__ void stats_begin(const f32x16& P, const RowStat& st, float c2, float& mn,
                                            float& nmc, float& corr) {
  const float a0 = max3(P[0], P[1], P[2]), a1 = max3(P[3], P[4], P[5]), a2 = max3(P[6], P[7], P[8]);
  const float a3 = max3(P[9], P[10], P[11]), a4 = max3(P[12], P[13], P[14]);
  mn = max3(max3(a0, a1, a2), max3(a3, a4, P[15]), st.m);
  nmc = -mn * c2;
  corr = ex2((st.m - mn) * c2);  // exactly 1 when the max did not move
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
constexpr float kRebase = 1.0e18f;

template <bool F32, int KS, int J>
__device__ __forceinline__ void stats_slot(f32x16& acc, const bf16x8 (&a)[KS], const bf16x8 (&b)[KS],
                                           const f32x16& P, float c2, float nmc, float (&x)[16], float& s0,
                                           float& s1) {
  using SL = Slots<KS>;
  if (J == 0) acc = f32x16{0};
  mfma_step<F32>(acc, a[J], b[J]);
  fence_sched();
  stats_stage_fma<SL::reduce(J), SL::reduce(J + 1)>(x, P, c2, nmc);
  if constexpr (J >= 1) stage_exp<SL::reduce(J - 1), SL::reduce(J)>(x);
  if constexpr (J >= 2) stage_add<SL::reduce(J - 2), SL::reduce(J - 1)>(x, s0, s1);
  fence_sched();
}

template <bool F32, int KS, int J = 0>
__device__ __forceinline__ void stats_slots(f32x16& acc, const bf16x8 (&a)[KS], const bf16x8 (&b)[KS],
                                            const f32x16& P, float c2, float nmc, float (&x)[16], float& s0,
                                            float& s1) {
  stats_slot<F32, KS, J>(acc, a, b, P, c2, nmc, x, s0, s1);
  if constexpr (J + 1 < KS) stats_slots<F32, KS, J + 1>(acc, a, b, P, c2, nmc, x, s0, s1);
}

__device__ __forceinline__ void stats_fold(const f32x16& P, RowStat& st, float c2);

// DEFER: the sum is taken as it is and only its running maximum over several units is kept in `worst`; the
// caller checks that once per key tile and, if it ever exceeded kRebase, redoes those units on the exact path.
template <bool F32, int KS, bool DEFER = false>
__device__ __forceinline__ void stats_unit(f32x16& acc, const bf16x8 (&a)[KS], const bf16x8 (&b)[KS],
                                           const f32x16& P, RowStat& st, float c2, float* worst = nullptr) {
  using SL = Slots<KS>;
  float s0 = 0.f, s1 = 0.f, x[16];
  const float nmc = -st.m * c2;
  stats_slots<F32, KS>(acc, a, b, P, c2, nmc, x, s0, s1);
  // drain the pipeline: last exp2 stage, last two sum stages
  stage_exp<SL::reduce(KS - 1), SL::reduce(KS)>(x);
  stage_add<SL::reduce(KS - 2), SL::reduce(KS - 1)>(x, s0, s1);
  stage_add<SL::reduce(KS - 1), SL::reduce(KS)>(x, s0, s1);
  const float D = st.D + (s0 + s1);
  if constexpr (DEFER) {
    st.D = D;  // +inf at worst (a row without a reference, or a logit 2^60 in weight above it): never NaN
    *worst = fmaxf(*worst, D);
  } else {
    if (__any(!(D <= kRebase))) stats_fold(P, st, c2);  // some row needs a new reference: exact path for the wave
    else st.D = D;
  }
  fence_sched();
}

// fold one finished tile into its row statistics, nothing to overlap with
__device__ __forceinline__ void stats_fold(const f32x16& P, RowStat& st, float c2) {
  float mn, nmc, corr;
  stats_begin(P, st, c2, mn, nmc, corr);
  const float s = (stats_group(P, 0, c2, nmc) + stats_group(P, 1, c2, nmc)) +
                  (stats_group(P, 2, c2, nmc) + stats_group(P, 3, c2, nmc));
  st.D = fmaf(st.D, corr, s);
  st.m = mn;
}

// Key tiles per split.  Where the heads have lengths of their own, often far below the bound that the plan was made
// for, every split takes its share of the head's own tiles; cut at the bound, the last splits were empty and part of
// the chip idle (64 heads of about 8000 of 13000 rows: 90 -> 62 us).
__device__ __forceinline__ int split_length(const Plan& pl, int tiles, int splits, int tiles_per_split) {
  return pl.n_ctx ? __builtin_amdgcn_readfirstlane((tiles + splits - 1) / splits) : tiles_per_split;
}

// NQ 32-row query sub-tiles per wave, NW waves per workgroup: 32*NQ*NW query rows per workgroup.
template <bool F32, int HD, int KS, int NQ, int NW>
__global__ __launch_bounds__(NW * 64, (NW == 1 || (HD > 128 && NW < 4) ? 1 : 2)) void score_stats(const bf16_t* __restrict__ q,
                                                          const bf16_t* __restrict__ k,
                                                          float2* __restrict__ stats, Plan pl) {
  using TL = Tile<HD>;
  using ST = Stager<HD, NW>;
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
  const int rb = blockIdx.x >> 3, split = blockIdx.y;
  const int bh = blockIdx.z * 8 + (blockIdx.x & 7);
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
  uint32_t koff[ST::kPer];
  const int last_chunk = pl.d / 8 - 1;
  ST::offsets(koff, wave, lane, kstride, last_chunk);

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
        mfma_chain<KS, F32>(accA, kf, qf[u % NQ]);
        stats_fold(accA, st[u % NQ], c2);
      }
      if (NQ == 1) read_frags<HD, KS>(kf, lds, 1, l32, hi);
      mfma_chain<KS, F32>(accB, kf, qf[NQ - 1]);
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
        stats_unit<F32, KS>(accA, kf, qf[0], accB, st[NQ - 1], c2);
        RowStat before[NQ];
#pragma unroll
        for (int s = 0; s < NQ; s++) before[s] = st[s];
        float worst = 0.f;
#pragma unroll
        for (int u = 1; u < 2 * NQ; u++) {
          const int s = u % NQ, sp = (u - 1) % NQ;
          if (u == NQ) read_frags<HD, KS>(kf, cur, 1, l32, hi);
          if (u & 1) stats_unit<F32, KS, true>(accB, kf, qf[s], accA, st[sp], c2, &worst);
          else       stats_unit<F32, KS, true>(accA, kf, qf[s], accB, st[sp], c2, &worst);
        }
        if (__any(!(worst <= kRebase))) {
#pragma unroll
          for (int s = 0; s < NQ; s++) st[s] = before[s];
#pragma unroll
          for (int u = 0; u < 2 * NQ - 1; u++) {
            if (u == 0 || u == NQ) read_frags<HD, KS>(kf, cur, u / NQ, l32, hi);
            mfma_chain<KS, F32>(accA, kf, qf[u % NQ]);
            stats_fold(accA, st[u % NQ], c2);
          }
        }
      } else {
#pragma unroll
        for (int u = 0; u < 2 * NQ; u++) {
          const int s = u % NQ, sp = (u + NQ * 2 - 1) % NQ;
          if (u == NQ) read_frags<HD, KS>(kf, cur, 1, l32, hi);
          if (u & 1) stats_unit<F32, KS>(accB, kf, qf[s], accA, st[sp], c2);
          else       stats_unit<F32, KS>(accA, kf, qf[s], accB, st[sp], c2);
        }
      }
    }
    wait_vmem();
    __syncthreads();
    buf ^= 1;
  }
  if (active) stats_fold(accB, st[NQ - 1], c2);  // last unit in flight (or the filler)

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
          mfma_chain<KS, F32>(acc, kf, qf[s]);
#pragma unroll
          for (int v = 0; v < 16; v++)
            if (ks * 32 + (v >> 2) * 8 + hi * 4 + (v & 3) >= nrows) acc[v] = kMasked;
          stats_fold(acc, st[s], c2);
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
            mfma_chain<KS, F32>(acc, kf, qf[s]);
#pragma unroll
            for (int v = 0; v < 16; v++)
              if (pt * kKeyTile + ks * 32 + (v >> 2) * 8 + hi * 4 + (v & 3) > t_row) acc[v] = kMasked;
            stats_fold(acc, st[s], c2);
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
    const float Dn = st[s].D * ex2((st[s].m - mn) * c2) + Do * ex2((mo - mn) * c2);
    const int r = row0 + s * 32 + l32;
    if (hi == 0 && r < pl.R)
      out[((size_t)bh * n_splits + split) * Rpad + r] = make_float2(mn * c2, Dn);
  }
}

// ------------------------------------------------------- between the passes
// A row's base-2 log-sum-exp from its key splits, for ROWS rows at a time (r0, r0 + step, ..; rows beyond R repeat the
// last one).  Eight splits of every row are loaded together.
template <int ROWS>
__device__ __forceinline__ void combine_splits(float (&lse)[ROWS], const float2* __restrict__ st, int r0, int step,
                                               const Plan& pl) {
  constexpr int kSplitsAtOnce = 8;
  float mx[ROWS], den[ROWS];
#pragma unroll
  for (int i = 0; i < ROWS; i++) mx[i] = kMasked, den[i] = 0.f;
  for (int s0 = 0; s0 < pl.n_splits; s0 += kSplitsAtOnce) {
    float2 e[ROWS][kSplitsAtOnce];
#pragma unroll
    for (int i = 0; i < ROWS; i++)
#pragma unroll
      for (int j = 0; j < kSplitsAtOnce; j++)
        e[i][j] = st[(size_t)min(s0 + j, pl.n_splits - 1) * pl.Rpad + min(r0 + i * step, pl.R - 1)];
#pragma unroll
    for (int i = 0; i < ROWS; i++) {
      float m = mx[i];
#pragma unroll
      for (int j = 0; j < kSplitsAtOnce; j++) m = fmaxf(m, e[i][j].x);
      float sum = den[i] * ex2(mx[i] - m);
#pragma unroll
      for (int j = 0; j < kSplitsAtOnce; j++)
        sum += s0 + j < pl.n_splits ? e[i][j].y * ex2(e[i][j].x - m) : 0.f;
      mx[i] = m, den[i] = sum;
    }
  }
#pragma unroll
  for (int i = 0; i < ROWS; i++) lse[i] = mx[i] + __log2f(den[i]);
}

// One thread per row, rows of a head dense.  Only where pass 2 runs over several rounds of workgroups (launch_rows).
__global__ void combine_row_stats(const float2* __restrict__ stats, float* __restrict__ lse, Plan pl, int total) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= total) return;
  const int bh = i / pl.R;
  float val[1];
  combine_splits<1>(val, stats + (size_t)bh * pl.n_splits * pl.Rpad, i - bh * pl.R, 0, pl);
  lse[i] = val[0];
}

// Fills LDS with what pass 2 adds to every scaled logit of a row: minus the row's base-2 log-sum-exp, from
// row_lse * lse_scale (the caller's natural-log normalisers, or combined ones) or, if that is null, from the key
// splits of pass 1; rows beyond R get -inf (weight 0).  In two parts: request() asks for the first rows ahead of the
// workgroup's other loads, finish() comes behind them, so that its wait is not for those (they return in order).
template <int THREADS, int ROWS>
struct NlseFill {
  float early[ROWS];  // rows threadIdx.x + i * THREADS

  __device__ __forceinline__ void request(const float* __restrict__ row_lse, int bh, const Plan& pl) {
    if (!row_lse) return;
#pragma unroll
    for (int i = 0; i < ROWS; i++) early[i] = row_lse[(size_t)bh * pl.R + min((int)threadIdx.x + i * THREADS, pl.R - 1)];
  }
  __device__ __forceinline__ void finish(float* nlse, int rows, const float2* __restrict__ stats,
                                         const float* __restrict__ row_lse, float lse_scale, int bh, const Plan& pl) {
    auto put = [&](int r, float lse) {
      if (r < rows) nlse[r] = r < pl.R ? -lse : -INFINITY;
    };
    if (row_lse) {
#pragma unroll
      for (int i = 0; i < ROWS; i++) put(threadIdx.x + i * THREADS, early[i] * lse_scale);
      for (int r = threadIdx.x + ROWS * THREADS; r < rows; r += THREADS)
        put(r, row_lse[(size_t)bh * pl.R + min(r, pl.R - 1)] * lse_scale);
      return;
    }
    for (int r0 = threadIdx.x; r0 < rows; r0 += 2 * THREADS) {
      float val[2];
      combine_splits<2>(val, stats + (size_t)bh * pl.n_splits * pl.Rpad, r0, THREADS, pl);
      put(r0, val[0]), put(r0 + THREADS, val[1]);
    }
  }
};

// ------------------------------------------------------------------ pass 2
// Column reduction of the previous accumulator tile (16 query rows of one key),
// sliced like the statistics above.  nl[v] = -(base-2 lse) of the value's row.
template <int REDUCE>
__device__ __forceinline__ float col_group(const f32x16& P, const float (&nl)[16], int g, float c2) {
  const float x0 = fmaf(P[4 * g + 0], c2, nl[4 * g + 0]), x1 = fmaf(P[4 * g + 1], c2, nl[4 * g + 1]);
  const float x2 = fmaf(P[4 * g + 2], c2, nl[4 * g + 2]), x3 = fmaf(P[4 * g + 3], c2, nl[4 * g + 3]);
  if (REDUCE == EPICACHE_REDUCE_MAX) return vmax(vmax3(x0, x1, x2), x3);
  return (ex2(x0) + ex2(x1)) + (ex2(x2) + ex2(x3));
}

template <int REDUCE>
__device__ __forceinline__ float col_merge(float col, float a, float b, float c, float d) {
  if (REDUCE == EPICACHE_REDUCE_MAX) return vmax3(vmax3(a, b, c), d, col);
  return col + ((a + b) + (c + d));
}

template <int LO, int HI>
__device__ __forceinline__ void col_stage_fma(float (&x)[16], const f32x16& P, const float (&nl)[16], float c2) {
#pragma unroll
  for (int v = LO; v < HI; v++) x[v] = fmaf(P[v], c2, nl[v]);
#pragma unroll
  for (int v = LO; v < HI; v++) pin(x[v]);
}

template <bool F32, int KS, int REDUCE, int J>
__device__ __forceinline__ void reduce_slot(f32x16& acc, const bf16x8 (&a)[KS], const bf16x8 (&b)[KS],
                                            const f32x16& P, const float (&nl)[16], float c2, float (&x)[16],
                                            float& s0, float& s1) {
  using SL = Slots<KS>;
  if (J == 0) acc = f32x16{0};
  mfma_step<F32>(acc, a[J], b[J]);
  fence_sched();
  col_stage_fma<SL::reduce(J), SL::reduce(J + 1)>(x, P, nl, c2);
  if constexpr (REDUCE == EPICACHE_REDUCE_MAX) {
    if constexpr (J >= 1) stage_max<SL::reduce(J - 1), SL::reduce(J)>(x, s0, s1);
  } else {
    if constexpr (J >= 1) stage_exp<SL::reduce(J - 1), SL::reduce(J)>(x);
    if constexpr (J >= 2) stage_add<SL::reduce(J - 2), SL::reduce(J - 1)>(x, s0, s1);
  }
  fence_sched();
}

template <bool F32, int KS, int REDUCE, int J = 0>
__device__ __forceinline__ void reduce_slots(f32x16& acc, const bf16x8 (&a)[KS], const bf16x8 (&b)[KS],
                                             const f32x16& P, const float (&nl)[16], float c2, float (&x)[16],
                                             float& s0, float& s1) {
  reduce_slot<F32, KS, REDUCE, J>(acc, a, b, P, nl, c2, x, s0, s1);
  if constexpr (J + 1 < KS) reduce_slots<F32, KS, REDUCE, J + 1>(acc, a, b, P, nl, c2, x, s0, s1);
}

// acc <- MFMA chain, interleaved with reducing P (the tile finished one unit earlier; nl = minus the
// base-2 log-sum-exp of each of its 16 rows) into `col`.
template <bool F32, int KS, int REDUCE>
__device__ __forceinline__ void reduce_unit(f32x16& acc, const bf16x8 (&a)[KS], const bf16x8 (&b)[KS],
                                            const f32x16& P, const float (&nl)[16], float& col, float c2) {
  using SL = Slots<KS>;
  float x[16];
  float s0 = REDUCE == EPICACHE_REDUCE_MAX ? -INFINITY : 0.f, s1 = s0;
  reduce_slots<F32, KS, REDUCE>(acc, a, b, P, nl, c2, x, s0, s1);
  if constexpr (REDUCE == EPICACHE_REDUCE_MAX) {
    stage_max<SL::reduce(KS - 1), SL::reduce(KS)>(x, s0, s1);
    col = vmax3(col, s0, s1);
  } else {
    stage_exp<SL::reduce(KS - 1), SL::reduce(KS)>(x);
    stage_add<SL::reduce(KS - 2), SL::reduce(KS - 1)>(x, s0, s1);
    stage_add<SL::reduce(KS - 1), SL::reduce(KS)>(x, s0, s1);
    col += s0 + s1;
  }
  fence_sched();
}

__device__ __forceinline__ void read_nlse(float (&nl)[16], const float* nlse, int row0, int hi) {
#pragma unroll
  for (int g4 = 0; g4 < 4; g4++) {
    const float4 x = *reinterpret_cast<const float4*>(nlse + row0 + g4 * 8 + hi * 4);
    nl[g4 * 4 + 0] = x.x, nl[g4 * 4 + 1] = x.y, nl[g4 * 4 + 2] = x.z, nl[g4 * 4 + 3] = x.w;
  }
}

// NK 32-key sub-tiles per wave (1 for rows of more than 128 elements: the registers), 4 waves.
template <bool F32, int HD, int KS, int NK, int REDUCE>
__global__ __launch_bounds__(256, 2) void score_reduce(const bf16_t* __restrict__ q,
                                                       const bf16_t* __restrict__ k,
                                                       const float2* __restrict__ stats,
                                                       const float* __restrict__ row_lse, float lse_scale,
                                                       float* __restrict__ scores, Plan pl) {
  using TL = Tile<HD>;
  constexpr int kKeys = 128 * NK;  // keys per workgroup
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  unsigned char* lds = smem;                                            // 2 query tiles
  float* nlse = reinterpret_cast<float*>(smem + 2 * TL::kTileBytes);    // [Rpad + 64] minus base-2 lse
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, hi = lane >> 5;
  // XCD-aware ids as in pass 1: the key blocks of one (b, h) all stream the same query rows through LDS
  // and are given ids that land on one XCD: id = xcd + 8 * (key block + NKB * (bh / 8)), bh % 8 = xcd.
  const int kb = blockIdx.x >> 3;
  const int bh = blockIdx.y * 8 + (blockIdx.x & 7);
  if (bh >= pl.nb * pl.Hkv) return;
  const int b = batch_of(pl, bh), h = bh - b * pl.Hkv;
  const int N = ctx_rows(pl, bh);
  if (kb * kKeys >= N) return;  // a shorter head of a ragged batch: no keys here
  const int key0 = kb * kKeys + wave * (32 * NK);
  const float c2 = pl.c2;

  using ST = Stager<HD, 4>;
  const unsigned char* qbase = reinterpret_cast<const unsigned char*>(q + b * pl.qsb + (int64_t)(h * pl.G) * pl.qsh);
  const size_t qsh = (size_t)pl.qsh * 2;
  const uint32_t qstride = (uint32_t)pl.qst * 2;
  const int p = pl.p, last_row = pl.R - 1;
  // In registers before the loop: a scalar load inside it or right in front of it shares its counter with the LDS
  // reads, which could then only be waited for all at once (pass 2 of 128 heads, R = 512, N = 8192: +4 %).
  float inv_p = pl.inv_p;
  float* out = scores + (size_t)bh * pl.N;
  asm volatile("" : "+s"(inv_p), "+s"(out));
  const bool dense_tiles = p % 64 == 0;  // every 64-row tile lies inside one query head
  uint32_t qoff[ST::kPer];
  const int last_chunk = pl.d / 8 - 1;
  ST::offsets(qoff, wave, lane, qstride, last_chunk);
  const uint32_t lds0 = lds_address(lds);
  // dense tiles are staged in order, so the address of the next one is carried along instead of being derived
  // from the tile index with a division per tile
  const unsigned char* qtile = qbase;  // first row of the next tile to stage
  int qtile_row = 0;                   // that row's index within its query head
  auto stage_queries = [&](uint32_t dst, int t) {
    if (dense_tiles) {
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
  stage_queries(lds0, 0);

  // every query row's normaliser, then 64 rows of -inf (the "tile before the first")
  NlseFill<256, 5> fill;
  fill.request(row_lse, bh, pl);

  // key fragments of this wave stay in registers for the whole query loop
  const bf16_t* kbase = k + b * pl.ksb + (int64_t)h * pl.ksh;
  bf16x8 kf[NK][KS];
#pragma unroll
  for (int s = 0; s < NK; s++)
    load_row_frags<KS>(kf[s], kbase + (int64_t)min(key0 + s * 32 + l32, N - 1) * pl.kst, hi, pl.d);

  fill.finish(nlse, pl.Rpad + 64, stats, row_lse, lse_scale, bh, pl);

  // The fragments are used here, i.e. loaded before the wait below.  Left to itself the compiler sinks these
  // loads behind the barrier, finds them outstanding at the loop's entry and puts a counted wait in front of the
  // first use of each inside the loop; from the second iteration on those waits only see the tile in flight and
  // make every wave wait for it a unit and a half after it was requested.
#pragma unroll
  for (int s = 0; s < NK; s++)
#pragma unroll
    for (int j = 0; j < KS; j++) asm volatile("" : "+v"(kf[s][j]));

  // SUM: running sum of weights.  MAX: running max of the base-2 log weight
  // (exp2 is monotone, so one exponential per key at the end is enough).
  float col[NK];
#pragma unroll
  for (int s = 0; s < NK; s++) col[s] = REDUCE == EPICACHE_REDUCE_MAX ? -INFINITY : 0.f;
  f32x16 accA, accB;
#pragma unroll
  for (int v = 0; v < 16; v++) accA[v] = accB[v] = 0.f;
  // "previous tile" of the very first unit: rows [Rpad, Rpad+64) of nlse are -inf, i.e. a no-op
  float nlP[16], nlC[16];

  wait_vmem();
  __syncthreads();  // query tile 0 and nlse[] are in LDS
  read_nlse(nlP, nlse, pl.Rpad, hi);

  const int qtiles = pl.Rpad / 64;
  int buf = 0;
  // Units of one query tile: (qs, s) for qs in {0,1} (32-row halves), s in {0,1} (key halves of the
  // wave): u = 2*qs + s accumulates into accA (u even) / accB (u odd) while unit u-1 is reduced.
  for (int t = 0; t < qtiles; t++) {
    const unsigned char* cur = lds + buf * TL::kTileBytes;
    if (t + 1 < qtiles) stage_queries(lds0 + (buf ^ 1) * TL::kTileBytes, t + 1);
    if constexpr (NK == 2) {
      bf16x8 qf0[KS], qf1[KS];
      read_frags<HD, KS>(qf0, cur, 0, l32, hi);
      read_frags<HD, KS>(qf1, cur, 1, l32, hi);
      read_nlse(nlC, nlse, t * 64, hi);
      // unit 0: rows qs=0, keys s=0; previous unit = (prev tile, qs=1, s=1) with nlP
      reduce_unit<F32, KS, REDUCE>(accA, qf0, kf[0], accB, nlP, col[1], c2);
      read_nlse(nlP, nlse, t * 64 + 32, hi);
      reduce_unit<F32, KS, REDUCE>(accB, qf0, kf[1], accA, nlC, col[0], c2);
      reduce_unit<F32, KS, REDUCE>(accA, qf1, kf[0], accB, nlC, col[1], c2);
      reduce_unit<F32, KS, REDUCE>(accB, qf1, kf[1], accA, nlP, col[0], c2);
    } else {
      bf16x8 qf[KS];
      read_frags<HD, KS>(qf, cur, 0, l32, hi);
      reduce_unit<F32, KS, REDUCE>(accA, qf, kf[0], accB, nlP, col[0], c2);
      read_nlse(nlC, nlse, t * 64, hi);
      read_frags<HD, KS>(qf, cur, 1, l32, hi);
      reduce_unit<F32, KS, REDUCE>(accB, qf, kf[0], accA, nlC, col[0], c2);
      read_nlse(nlP, nlse, t * 64 + 32, hi);
    }
    wait_vmem();
    __syncthreads();
    buf ^= 1;
  }
  {  // drain: last unit (qs=1, s=1) sits in accB with nlP
    const float s0 = col_group<REDUCE>(accB, nlP, 0, c2), s1 = col_group<REDUCE>(accB, nlP, 1, c2);
    const float s2 = col_group<REDUCE>(accB, nlP, 2, c2), s3 = col_group<REDUCE>(accB, nlP, 3, c2);
    col[NK - 1] = col_merge<REDUCE>(col[NK - 1], s0, s1, s2, s3);
  }

#pragma unroll
  for (int s = 0; s < NK; s++) {
    // lanes l and l^32 hold the same key over disjoint query rows
    const float o = __shfl_xor(col[s], 32);
    float val;
    if (REDUCE == EPICACHE_REDUCE_MAX) val = ex2(fmaxf(col[s], o));
    else val = col[s] + o;
    const int key = key0 + s * 32 + l32;
    if (hi == 0 && key < N) out[key] = val;
  }
}

// ------------------------------------------------------- pass 2, streaming form
// For R <= 256 (all query rows of a KV head fit one workgroup): same data flow as pass 1 - query
// fragments stay in registers, 64-key tiles stream through LDS - with the operands swapped so that
// a lane owns one key column and 16 query rows.  Each wave reduces its own rows; the per-key
// partial results of the NW waves meet in LDS once per tile.  Reads K with fully coalesced
// 1 KiB bursts, which the key-stationary form above cannot do when R is small.
template <int KS, int REDUCE>
__device__ __forceinline__ void col_fold(const f32x16& P, const float (&nl)[16], float& col, float c2) {
  const float s0 = col_group<REDUCE>(P, nl, 0, c2), s1 = col_group<REDUCE>(P, nl, 1, c2);
  const float s2 = col_group<REDUCE>(P, nl, 2, c2), s3 = col_group<REDUCE>(P, nl, 3, c2);
  col = col_merge<REDUCE>(col, s0, s1, s2, s3);
}

template <bool F32, int HD, int KS, int NQ, int NW, int REDUCE>
__global__ __launch_bounds__(NW * 64, (NW == 1 || (HD > 128 && NW < 4) ? 1 : 2)) void score_reduce_stream(const bf16_t* __restrict__ q,
                                                                  const bf16_t* __restrict__ k,
                                                                  const float2* __restrict__ stats,
                                                                  const float* __restrict__ row_lse, float lse_scale,
                                                                  float* __restrict__ scores, Plan pl) {
  using TL = Tile<HD>;
  using ST = Stager<HD, NW>;
  constexpr int kRows = 32 * NQ * NW;
  constexpr float kNeutral = REDUCE == EPICACHE_REDUCE_MAX ? -INFINITY : 0.f;
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  unsigned char* lds = smem;                                             // 2 key tiles
  float* nlse = reinterpret_cast<float*>(smem + 2 * TL::kTileBytes);     // [kRows]
  float(*part)[NW][64] = reinterpret_cast<float(*)[NW][64]>(nlse + kRows);  // [2]
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, hi = lane >> 5;
  const int split = blockIdx.x >> 3, bh = blockIdx.y * 8 + (blockIdx.x & 7);  // a head's splits on one XCD, as above
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
  if (t_begin >= t_end) return;  // a shorter head of a ragged batch: no keys in this split

  const unsigned char* kbase = reinterpret_cast<const unsigned char*>(k + b * pl.ksb + (int64_t)h * pl.ksh);
  const uint32_t kstride = (uint32_t)pl.kst * 2;
  uint32_t koff[ST::kPer];
  const int last_chunk = pl.d / 8 - 1;
  ST::offsets(koff, wave, lane, kstride, last_chunk);
  const uint32_t lds0 = lds_address(lds);
  auto stage_keys = [&](uint32_t dst, int t) {
    const unsigned char* tile = kbase + (size_t)t * kKeyTile * kstride;
    const int nrows = N - t * kKeyTile;
    if (nrows >= kKeyTile) ST::run(dst, tile, koff, wave);
    else  // ragged last tile: rows beyond N re-read the last key; their results are never written
      ST::run_rows(dst, wave, lane, [=](int row) { return tile + (size_t)min(row, nrows - 1) * kstride; }, last_chunk);
  };
  stage_keys(lds0, t_begin);

  NlseFill<NW * 64, (kRows + NW * 64 - 1) / (NW * 64)> fill;
  fill.request(row_lse, bh, pl);

  // query fragments (A operand: rows = queries) stay in registers for the whole key loop; rows beyond R have weight 0
  bf16x8 qf[NQ][KS];
#pragma unroll
  for (int s = 0; s < NQ; s++) {
    int g, t;
    head_and_token(pl.p, pl.inv_p, min(row0 + s * 32 + l32, pl.R - 1), g, t);
    load_row_frags<KS>(qf[s], q + b * pl.qsb + (int64_t)(h * pl.G + g) * pl.qsh + (int64_t)t * pl.qst, hi, pl.d);
  }

  fill.finish(nlse, kRows, stats, row_lse, lse_scale, bh, pl);

  wait_vmem();
  __syncthreads();  // first key tile and nlse[] are in LDS

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
      const float v = REDUCE == EPICACHE_REDUCE_MAX ? fmaxf(lo, up) : lo + up;
      if (hi == 0) part[t & 1][wave][ks * 32 + l32] = v;
    }
  };
  auto write_scores = [&](int t) {  // after the barrier that completes part[t & 1]
    if (tid < 64) {
      const int key = t * kKeyTile + tid;
      if (key < N) {
        float v = part[t & 1][0][tid];
#pragma unroll
        for (int w = 1; w < NW; w++)
          v = REDUCE == EPICACHE_REDUCE_MAX ? fmaxf(v, part[t & 1][w][tid]) : v + part[t & 1][w][tid];
        scores[(size_t)bh * pl.N + key] = REDUCE == EPICACHE_REDUCE_MAX ? ex2(v) : v;
      }
    }
  };

  int buf = 0;
  f32x16 accA, accB;                             // accB after a tile: its last unit, still to be reduced
#pragma unroll
  for (int v = 0; v < 16; v++) accB[v] = kMasked;  // before the first tile: a filler whose weights are 0; what it
                                                   // leaves in cs_prev is never exchanged
  float cs_prev[2] = {kNeutral, kNeutral};       // partials of the previous tile (keys ks*32 + l32)
  for (int t = t_begin; t < t_end; t++) {
    const unsigned char* cur = lds + buf * TL::kTileBytes;
    if (t + 1 < t_end) stage_keys(lds0 + (buf ^ 1) * TL::kTileBytes, t + 1);
    float cs[2] = {kNeutral, kNeutral};  // this wave's rows, keys ks*32 + l32 of the tile
    if (active) {
      // units (ks, s): key half ks, query sub-tile s; unit u accumulates into accA/accB (u even/odd)
      // while unit u-1 is reduced over its 16 rows into cs[ks of u-1]
      bf16x8 kf[KS];
      read_frags<HD, KS>(kf, cur, 0, l32, hi);
#pragma unroll
      for (int u = 0; u < 2 * NQ; u++) {
        const int s = u % NQ, sp = (u + 2 * NQ - 1) % NQ, ksp = (u - 1) / NQ;
        if (u == NQ) read_frags<HD, KS>(kf, cur, 1, l32, hi);
        float nl[16];  // minus lse of the 16 rows this lane holds of the previous unit
        read_nlse(nl, nlse, row0 + sp * 32, hi);
        if (u == 0) {
          reduce_unit<F32, KS, REDUCE>(accA, qf[0], kf, accB, nl, cs_prev[1], c2);  // last unit of tile t-1
        } else if (u & 1) {
          reduce_unit<F32, KS, REDUCE>(accB, qf[s], kf, accA, nl, cs[ksp], c2);
        } else {
          reduce_unit<F32, KS, REDUCE>(accA, qf[s], kf, accB, nl, cs[ksp], c2);
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
    float nl[16];
    read_nlse(nl, nlse, row0 + (NQ - 1) * 32, hi);
    col_fold<KS, REDUCE>(accB, nl, cs_prev[1], c2);  // last unit of the last tile: odd index, key half 1
  }
  exchange(cs_prev, t_end - 1);
  __syncthreads();
  write_scores(t_end - 1);
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

template <bool F32, int HD, int KS, int NQ, int NW>
hipError_t launch_rows(const Plan& pl, const bf16_t* q, const bf16_t* k, float* scores, float2* stats,
                       const float* row_lse, hipStream_t stream) {
  using TL = Tile<HD>;
  const int bh8 = (pl.nb * pl.Hkv + 7) / 8;  // ids whose bh falls beyond the batch exit at once
  if (!row_lse) {
    const int n_rb = (pl.R + 32 * NQ * NW - 1) / (32 * NQ * NW);
    hipLaunchKernelGGL((score_stats<F32, HD, KS, NQ, NW>), dim3(8 * n_rb, pl.n_splits, bh8), dim3(NW * 64), 0, stream, q, k,
                       stats, pl);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  float lse_scale = 1.44269504088896340736f;
  if (pl.R <= pl.stats_rows_per_wg) {
    const dim3 grid(8 * pl.reduce_splits, bh8);
    const size_t smem = 2 * TL::kTileBytes + (32 * NQ * NW + 2 * NW * 64) * sizeof(float);
    if (pl.reduce == EPICACHE_REDUCE_MAX)
      return launch_lds(score_reduce_stream<F32, HD, KS, NQ, NW, EPICACHE_REDUCE_MAX>, grid, NW * 64, smem, stream, q, k,
                        stats, row_lse, lse_scale, scores, pl);
    return launch_lds(score_reduce_stream<F32, HD, KS, NQ, NW, EPICACHE_REDUCE_SUM>, grid, NW * 64, smem, stream, q, k, stats,
                      row_lse, lse_scale, scores, pl);
  }
  constexpr int NK = HD > 128 ? 1 : 2;
  const int key_blocks = (pl.N + 128 * NK - 1) / (128 * NK);
  // The key splits become one number per row in every workgroup of pass 2 while its keys are on their way, or, where
  // the chip takes more than one round of those workgroups, in a kernel of its own: 5 us and a launch, against 2 us per
  // round (64 heads of 512 rows, 8192 keys, 4 rounds: pass 2 80 -> 89 us).  The streaming form above always has one
  // round (32 heads of 192 rows, 4096 keys: 8.0 + 14.8 us with the kernel in between, 14.9 us without).
  if (!row_lse && (int64_t)key_blocks * pl.nb * pl.Hkv > 2 * 256) {
    float* lse = reinterpret_cast<float*>(stats + (size_t)pl.nb * pl.Hkv * pl.n_splits * pl.Rpad);
    const int total = pl.nb * pl.Hkv * pl.R;
    hipLaunchKernelGGL(combine_row_stats, dim3((total + 255) / 256), dim3(256), 0, stream, stats, lse, pl, total);
    row_lse = lse;
    lse_scale = 1.0f;
  }
  const dim3 grid(8 * key_blocks, bh8);
  const size_t smem = 2 * TL::kTileBytes + (size_t)(pl.Rpad + 64) * sizeof(float);
  if (pl.reduce == EPICACHE_REDUCE_MAX)
    return launch_lds(score_reduce<F32, HD, KS, NK, EPICACHE_REDUCE_MAX>, grid, 256, smem, stream, q, k, stats, row_lse,
                      lse_scale, scores, pl);
  return launch_lds(score_reduce<F32, HD, KS, NK, EPICACHE_REDUCE_SUM>, grid, 256, smem, stream, q, k, stats, row_lse,
                    lse_scale, scores, pl);
}

// Rows per workgroup of pass 1 (and of pass 2's streaming form) as make_plan chose them.
template <bool F32, int HD, int KS>
hipError_t launch_hd(const Plan& pl, const bf16_t* q, const bf16_t* k, float* scores, float2* stats,
                     const float* row_lse, hipStream_t stream) {
  if constexpr (HD <= 128 && !F32) {
    switch (pl.stats_rows_per_wg) {
      case 256: return launch_rows<F32, HD, KS, 2, 4>(pl, q, k, scores, stats, row_lse, stream);
      case 192: return launch_rows<F32, HD, KS, 3, 2>(pl, q, k, scores, stats, row_lse, stream);
    }
  }
  switch (pl.stats_rows_per_wg) {
    case 128: return launch_rows<F32, HD, KS, 1, 4>(pl, q, k, scores, stats, row_lse, stream);
    case 64: return launch_rows<F32, HD, KS, 1, 2>(pl, q, k, scores, stats, row_lse, stream);
    default: return launch_rows<F32, HD, KS, 1, 1>(pl, q, k, scores, stats, row_lse, stream);
  }
}

// Row layout in LDS and 32-byte steps of the contraction; row lengths in between are padded with zeros.
template <bool F32>
hipError_t launch_rows_of(const Plan& pl, const bf16_t* q, const bf16_t* k, float* scores, float2* stats,
                          const float* row_lse, hipStream_t stream) {
  if (pl.d <= 32) return launch_hd<F32, 64, 2>(pl, q, k, scores, stats, row_lse, stream);
  if (pl.d <= 64) return launch_hd<F32, 64, 4>(pl, q, k, scores, stats, row_lse, stream);
  if (pl.d <= 96) return launch_hd<F32, 128, 6>(pl, q, k, scores, stats, row_lse, stream);
  if (pl.d <= 128) return launch_hd<F32, 128, 8>(pl, q, k, scores, stats, row_lse, stream);
  if (pl.d <= 192) return launch_hd<F32, 256, 12>(pl, q, k, scores, stats, row_lse, stream);
  return launch_hd<F32, 256, 16>(pl, q, k, scores, stats, row_lse, stream);
}

}  // namespace

hipError_t launch_score_mfma(const Plan& pl, const void* q, const void* k, float* scores, float2* stats,
                             const float* row_lse, hipStream_t stream) {
  const bf16_t* qq = static_cast<const bf16_t*>(q);
  const bf16_t* kk = static_cast<const bf16_t*>(k);
  if (pl.dtype == EPICACHE_DTYPE_BF16) return launch_rows_of<false>(pl, qq, kk, scores, stats, row_lse, stream);
  // fp32 rows are moved as rows of twice as many two-byte units
  Plan p2 = pl;
  p2.d *= 2;
  for (int64_t* s : {&p2.qsb, &p2.qsh, &p2.qst, &p2.ksb, &p2.ksh, &p2.kst}) *s *= 2;
  return launch_rows_of<true>(p2, qq, kk, scores, stats, row_lse, stream);
}

}  // namespace epicache

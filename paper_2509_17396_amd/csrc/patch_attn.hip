// Attention output of the patch tokens (paper Sec. 2.3: the patched prompt is appended after the block and
// attends back to it): for every patch query t of every query head,
//   O_t = sum_i softmax_i(scale * q_t . k_i) v_i,   lse_t = log sum_i exp(scale * q_t . k_i),
// over the N context rows and, with causal_patch, the patch rows 0..t that follow them in K and V.
// The normalisers are exactly what the single-pass scoring takes, so this call followed by the scoring on
// supplied normalisers is the patch's whole pass through the layer plus Eq. 1.
//
// bf16, head_dim up to 128: one wave owns 32 query rows; tiles of 32 or 64 keys of K and of V stream HBM -> LDS
// (direct loads, double buffered).  Per 32-key half: S^T = K Q^T on the matrix cores (a lane owns one query
// column and 16 keys, as in the scoring statistics pass), an online softmax whose row maximum is shared by
// the two lanes of a row, and O^T += V^T P^T.  The V^T operand (8 consecutive
// keys of one head_dim column per lane) comes out of the row-major V tile with the transposing LDS load:
// 16 lanes that point at 4 keys x 16 columns get, lane i, the 4 keys of column i.
// The eight waves of a workgroup are RW blocks of 32 query rows times KW groups that take every KW-th tile of keys and
// merge their outputs at the end: few heads or few rows still fill the CU.  Where the heads are too few for the chip and the
// caller has room for it, several workgroups share the keys of a row (key splits): each leaves its output, reference and
// sum, and merge_attention puts them together.  8 heads of 256 rows, 18363 keys: 64 workgroups took some 200 us, 256 take 33.5
// and the merge 7.2.
// Weights: rounded to bf16 for head_dim 128; for other head dims cut into three bf16 parts whose sum is the fp32
// weight, so that the product with V is the fp32 one (12 instead of 4 MFMAs per 32 x 32 x 32 block).
// Anything else (fp32 inputs, head dims beyond 128): a plain fp32 kernel.
//
// The matrix products run over keys that a row does not see (weight 0), over parts of a weight that can be 0 and over
// the padding of a key row (0 in the query), so an infinity or a NaN there would make NaN of rows that it has no part in.
// It always shows in the sums: where one is not finite the workgroup goes through the keys a second time, counting the
// infinities and NaNs that each row does see apart from the finite values (add_not_finite).
#include <hip/hip_bf16.h>

#include <type_traits>

#include "launch_rules.h"
#include "mfma_tiles.h"

namespace epicache {
namespace {

typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(4))) short s16x4;

constexpr float kLazyBits = 8.f;

// V tiles use their own swizzle: 16-byte chunk c of key row r sits at position c ^ swz_v(r), so the four
// key rows that one transposing load touches fall into different 64-byte bank groups.
template <int HD>
__device__ __forceinline__ int swz_v(int r) { return HD == 64 ? 4 * (r & 1) : 4 * (r & 3); }

// Staging of one TK-row tile by NW waves, 1 KiB slabs; wave w takes slabs w, w + NW, ..  Full tiles go through a
// uniform slab address and a lane offset that only depends on the slab through the swizzle.
template <int HD, int NW, int TK, bool IS_V>
struct TileStager {
  using TL = Tile<HD>;
  static constexpr int kSlabs = TK * TL::kRowBytes / 1024;
  static constexpr int kPer = (kSlabs + NW - 1) / NW;
  // the swizzle repeats after this many rows; kOffsets slabs of a wave differ in it
  static constexpr int kPeriodRows = IS_V ? 4 : 16;
  static constexpr int kStepRows = NW * TL::kRowsPerSlab;  // rows from one slab of a wave to its next
  static constexpr int kOffsets = kStepRows >= kPeriodRows ? 1
                                  : kPeriodRows / kStepRows < kPer ? kPeriodRows / kStepRows : kPer;
  __device__ static __forceinline__ int chunk(int row, int lane, int last_chunk) {
    return min((lane % TL::kChunks) ^ (IS_V ? swz_v<HD>(row) : TL::swz(row)), last_chunk);
  }
  __device__ static __forceinline__ void offsets(uint32_t (&off)[kOffsets], int wave, int lane, uint32_t stride,
                                                 int last_chunk) {
#pragma unroll
    for (int i = 0; i < kOffsets; i++) {
      const int row = (wave + i * NW) * TL::kRowsPerSlab + lane / TL::kChunks;
      off[i] = lane / TL::kChunks * stride + chunk(row, lane, last_chunk) * 16;
    }
  }
  __device__ static __forceinline__ void run(uint32_t lds_tile, const unsigned char* tile, uint32_t stride,
                                             const uint32_t (&off)[kOffsets], int wave) {
#pragma unroll
    for (int i = 0; i < kPer; i++)
      if (kSlabs % NW == 0 || wave + i * NW < kSlabs) {
        const int slab = wave + i * NW;
        dma16_uniform_base(lds_tile + slab * 1024, tile + (size_t)(slab * TL::kRowsPerSlab) * stride, off[i % kOffsets]);
      }
  }
  // rows beyond the last one of a partial tile re-read it
  __device__ static __forceinline__ void run_tail(uint32_t lds_tile, const unsigned char* tile, uint32_t stride,
                                                  int nrows, int wave, int lane, int last_chunk) {
#pragma unroll
    for (int i = 0; i < kPer; i++)
      if (kSlabs % NW == 0 || wave + i * NW < kSlabs) {
        const int slab = wave + i * NW;
        const int row = slab * TL::kRowsPerSlab + lane / TL::kChunks;
        dma16_lane_ptr(lds_tile + slab * 1024,
                       tile + (size_t)min(row, nrows - 1) * stride + chunk(row, lane, last_chunk) * 16);
      }
  }
};

// A operand of O^T += V^T P^T for head_dim block `dblk` (32 columns) and the 16-key step `kstep` of the
// 32-key half `ks`: lane (m = l % 32, hi = l / 32) needs keys {4 hi .. 4 hi + 3} and {8 + 4 hi .. 8 + 4 hi + 3}
// (+ 16 kstep + 32 ks) of column 32 dblk + m, the key order in which the softmax weights sit in the lane.
template <int HD>
__device__ __forceinline__ bf16x8 read_vt_frag(const unsigned char* vtile, int ks, int kstep, int dblk, int lane) {
  const int s = lane & 15, gh = (lane >> 4) & 1, hi = lane >> 5;
  const int chunk = 4 * dblk + 2 * gh + ((s & 3) >> 1);      // 16-byte chunk of the row this lane points into
  const int half = (s & 1) * 8;
  s16x4 part[2];
#pragma unroll
  for (int g = 0; g < 2; g++) {
    const int row = 32 * ks + 16 * kstep + 8 * g + 4 * hi + (s >> 2);
    const unsigned char* p = vtile + row * Tile<HD>::kRowBytes + ((chunk ^ swz_v<HD>(row)) * 16) + half;
    part[g] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)LDS_PTR(p));
  }
  typedef __attribute__((ext_vector_type(8))) short s16x8;
  const s16x8 both = {part[0][0], part[0][1], part[0][2], part[0][3], part[1][0], part[1][1], part[1][2], part[1][3]};
  return __builtin_bit_cast(bf16x8, both);
}

// Eight fp32 weights as PARTS bf16 operands: rounded to one, or cut into three (8 + 8 + 8 bits of the significand)
// whose sum is exact.
template <int PARTS>
__device__ __forceinline__ void weight_frags(bf16x8 (&p)[PARTS], const float* e) {
  typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;
  if constexpr (PARTS == 1) {
    u32x4 packed;
#pragma unroll
    for (int j = 0; j < 4; j++) {
      const f32x2 pair = {e[2 * j], e[2 * j + 1]};
      packed[j] = __builtin_bit_cast(unsigned int, __builtin_convertvector(pair, bf16x2));
    }
    p[0] = __builtin_bit_cast(bf16x8, packed);
  } else {
    u32x4 packed[PARTS];
#pragma unroll
    for (int j = 0; j < 4; j++) {
      float a = e[2 * j], b = e[2 * j + 1];
#pragma unroll
      for (int i = 0; i < PARTS; i++) {
        const unsigned int ua = __float_as_uint(a), ub = __float_as_uint(b);
        packed[i][j] = __builtin_amdgcn_perm(ub, ua, 0x07060302);  // the upper halves, b's above a's
        a -= __uint_as_float(ua & 0xffff0000u), b -= __uint_as_float(ub & 0xffff0000u);
      }
    }
#pragma unroll
    for (int i = 0; i < PARTS; i++) p[i] = __builtin_bit_cast(bf16x8, packed[i]);
  }
}

// What the infinities and NaNs among the values add to one 32 x 32 block of O^T, for 16 keys: v as read from V, keys
// key + 0 .. 3 and key + 8 .. 11, of which the lane's row sees those up to last_key, w their weights.  Whether a row sees
// one of a kind is a product of zeros and ones.
// As in a sum of w * v: +inf, -inf, or NaN for both, for a NaN and for a weight that has underflowed to 0.
// Leaves the finite values in v.
__device__ __forceinline__ void add_not_finite(f32x16& o, bf16x8& v, int key, int last_key, const float* w) {
  typedef __attribute__((ext_vector_type(8))) unsigned short u16x8;
  constexpr unsigned short kOne = 0x3f80;
  u16x8 bits = __builtin_bit_cast(u16x8, v);
  bool none = true;
#pragma unroll
  for (int j = 0; j < 8; j++) none = none && (bits[j] & 0x7f80) != 0x7f80;
  if (__all(none)) return;
  auto add = [&](auto is_kind, auto counts, float what) {
    u16x8 a, b;
#pragma unroll
    for (int j = 0; j < 8; j++) a[j] = is_kind(bits[j]) ? kOne : 0, b[j] = key + (j & 3) + (j >> 2) * 8 <= last_key && counts(w[j]) ? kOne : 0;
    f32x16 n = f32x16{0};
    n = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), n, 0, 0, 0);
#pragma unroll
    for (int i = 0; i < 16; i++) o[i] += n[i] > 0.f ? what : 0.f;
  };
  add([](unsigned short x) { return x == 0x7f80; }, [](float x) { return x > 0.f; }, INFINITY);
  add([](unsigned short x) { return x == 0xff80; }, [](float x) { return x > 0.f; }, -INFINITY);
  add([](unsigned short x) { return (x & 0x7f80) == 0x7f80; }, [](float x) { return !(x > 0.f); }, NAN);
  add([](unsigned short x) { return (x & 0x7fff) > 0x7f80; }, [](float) { return true; }, NAN);
#pragma unroll
  for (int j = 0; j < 8; j++)
    if ((bits[j] & 0x7f80) == 0x7f80) bits[j] = 0;
  v = __builtin_bit_cast(bf16x8, bits);
}

// max(x[l], x[l ^ 32]) in every lane, on the vector ALU: the swap leaves the lower half's values in both
// halves of one register and the upper half's in both halves of the other.
__device__ __forceinline__ float max_across_halves(float x) {
  const unsigned int u = __float_as_uint(x);
  const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// The row maximum is taken with compiler-visible max operations, not the hand-written v_max3_f32 of the scoring
// kernels: the compiler's hazard pass does not treat inline assembly as a vector ALU instruction, so a
// hand-written v_max3_f32 scheduled straight behind the S chain read the accumulators before the matrix core
// had written them (no wait states inserted).  The stale maximum is still a valid reference, so results stayed
// inside the tolerance but differed from run to run in the last bf16 bit.
template <int HD, int TK>
constexpr size_t attention_group_lds() { return (size_t)4 * TK * Tile<HD>::kRowBytes; }  // K and V, two buffers each

// HD: row layout; KS 16-element steps of Q K^T; DB 32-column blocks of the output; PARTS: see weight_frags.
template <int HD, int KS, int DB, int PARTS, int RW, int KW, int TK>
__global__ __launch_bounds__(RW * KW * 64, RW * KW == 8 ? 2 : 1) void patch_attention_mfma(
    const bf16_t* __restrict__ q, const bf16_t* __restrict__ k, const bf16_t* __restrict__ v, bf16_t* __restrict__ out,
    float* __restrict__ lse_out, float* __restrict__ records, int key_splits, int split_keys, Plan pl) {
  using TL = Tile<HD>;
  using SK = TileStager<HD, RW, TK, false>;
  using SV = TileStager<HD, RW, TK, true>;
  constexpr int kTile = TK * TL::kRowBytes;
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int group = wave / RW, rwave = wave % RW;
  const int l32 = lane & 31, hi = lane >> 5;
  // XCD-aware ids: the row blocks of one (b, h) and key split read the same K and V and land on one XCD
  const int n_rb = gridDim.x >> 3, rb = blockIdx.x >> 3;
  const int unit = blockIdx.y * 8 + (blockIdx.x & 7);
  if (unit >= pl.nb * pl.Hkv * key_splits) return;
  const int bh = key_splits == 1 ? unit : unit / key_splits, split = unit - bh * key_splits;
  const int b = batch_of(pl, bh), h = bh - b * pl.Hkv;
  // the 32-row blocks are dealt evenly to the n_rb workgroups of a head: workgroups that do the same amount of
  // work stream K and V at the same pace, so the second one finds the tiles in the XCD's L2
  const int blocks_per_rb = ((pl.R + 31) / 32 + n_rb - 1) / n_rb;
  const int row0 = (rb * blocks_per_rb + rwave) * 32;
  const bool active = rwave < blocks_per_rb && row0 < pl.R;  // waves without rows only help staging the tiles
  const float c2 = pl.c2;
  const int N = ctx_rows(pl, bh);  // this head's own context length in a ragged batch
  const int n_keys = N + (pl.causal_patch ? pl.p : 0);  // context rows, then the patch's own rows
  const int first_tile = split * (split_keys / TK);
  const int tiles = key_splits == 1 ? (n_keys + TK - 1) / TK : min((n_keys + TK - 1) / TK, first_tile + split_keys / TK);

  const int r = row0 + l32;            // this lane's query row
  const bool row_ok = r < pl.R;
  int g_row, t_row;                    // query head of the group, patch token: sees patch keys 0..t_row
  head_and_token(pl.p, pl.inv_p, min(r, pl.R - 1), g_row, t_row);
  const int last_key = pl.causal_patch ? N + t_row : N - 1;  // the last one this row sees; it sees all before it
  const size_t orow = ((size_t)b * pl.Hq + h * pl.G + g_row) * pl.p + t_row;
  if (n_keys == 0) {  // a head without a single key (workgroup-uniform): O = 0, lse = -inf
    if (active && row_ok && group == 0) {
      if (hi == 0) lse_out[orow] = -INFINITY;
      for (int j = hi; j < pl.d / 8; j += 2) reinterpret_cast<uint4*>(out + orow * pl.d)[j] = make_uint4(0, 0, 0, 0);
    }
    return;
  }
  bf16x8 qf[KS];
  load_row_frags<KS>(qf, q + b * pl.qsb + (int64_t)(h * pl.G + g_row) * pl.qsh + (int64_t)t_row * pl.qst, hi, pl.d);

  const unsigned char* kbase = reinterpret_cast<const unsigned char*>(k + b * pl.ksb + (int64_t)h * pl.ksh);
  const unsigned char* vbase = reinterpret_cast<const unsigned char*>(v + b * pl.ksb + (int64_t)h * pl.ksh);
  const uint32_t kstride = (uint32_t)pl.kst * 2;
  const int last_chunk = pl.d / 8 - 1;
  unsigned char* const mine = smem + group * attention_group_lds<HD, TK>();  // this key group's tiles: K, K, V, V
  const uint32_t lds0 = lds_address(smem) + group * (uint32_t)attention_group_lds<HD, TK>();
  uint32_t koff[SK::kOffsets], voff[SV::kOffsets];
  SK::offsets(koff, rwave, lane, kstride, last_chunk);
  SV::offsets(voff, rwave, lane, kstride, last_chunk);
  auto stage = [&](int buf, int t) {
    const unsigned char* kt = kbase + (size_t)t * TK * kstride;
    const unsigned char* vt = vbase + (size_t)t * TK * kstride;
    const int nrows = n_keys - t * TK;
    if (nrows >= TK) {
      SK::run(lds0 + buf * kTile, kt, kstride, koff, rwave);
      SV::run(lds0 + (2 + buf) * kTile, vt, kstride, voff, rwave);
    } else if (nrows > 0) {
      SK::run_tail(lds0 + buf * kTile, kt, kstride, nrows, rwave, lane, last_chunk);
      SV::run_tail(lds0 + (2 + buf) * kTile, vt, kstride, nrows, rwave, lane, last_chunk);
    }
  };
  auto tile_ready = [&]() {
    wait_vmem();
    if constexpr (RW > 1) __syncthreads();
    else asm volatile("" ::: "memory");  // one wave per key group: the tiles are its own
  };

  f32x16 o[DB];  // O^T: head_dim block x 16 values (head_dim (v/4)*8 + hi*4 + v%4 of the block), this lane's row
  const float lazy = kLazyBits / c2;  // in units of the raw dot product
  float m, l;  // running row maximum (raw dot products, shared by lanes l and l^32) and this lane's sum

  const int steps = (tiles - first_tile + KW - 1) / KW;  // tile of step i: first_tile + i * KW + group
  // One tile out of buffer BUF.  The buffer index is a compile-time constant (the tile loop below is
  // unrolled by two) so that every LDS address is a loop-invariant lane offset plus an immediate.
  // CAREFUL: infinities and NaNs apart from the finite values; short of registers, not of time.
  auto tile_step = [&](auto buf_c, auto careful_c, int step) {
    const int BUF = buf_c;
    constexpr bool CAREFUL = decltype(careful_c)::value;
    constexpr int kUnroll = CAREFUL ? 1 : TK / 32;
    const unsigned char* ktile = mine + BUF * kTile;
    const unsigned char* vtile = mine + (2 + BUF) * kTile;
    const int t = first_tile + step * KW + group;
    if (step + 1 < steps) stage(BUF ^ 1, t + KW);
    if (active && t < tiles) {
      const int first = t * TK;
      const bool plain = first + TK <= N;  // every key of the tile is a context key: no masking
      bf16x8 kf[KS];
      if constexpr (!CAREFUL) read_frags<HD, KS>(kf, ktile, 0, l32, hi);
#pragma unroll kUnroll
      for (int ks = 0; ks < TK / 32; ks++) {
        f32x16 sacc;
        if constexpr (CAREFUL) {
          read_frags<HD, KS>(kf, ktile, ks, l32, hi);
#pragma unroll
          for (int j = 0; j < KS; j++)
            if (2 * j + hi > last_chunk) kf[j] = as_frag(make_uint4(0, 0, 0, 0));
        }
        mfma_chain<KS>(sacc, kf, qf);
        // LDS reads that the arithmetic below can hide: the key fragments of the second half and the
        // V^T fragments of this half
        if (!CAREFUL && ks + 1 < TK / 32) read_frags<HD, KS>(kf, ktile, 1, l32, hi);
        bf16x8 vf[DB][2];
        if constexpr (!CAREFUL) {
#pragma unroll
          for (int d = 0; d < DB; d++)
#pragma unroll
            for (int st = 0; st < 2; st++) vf[d][st] = read_vt_frag<HD>(vtile, ks, st, d, lane);
        }
        if (!plain) {
#pragma unroll
          for (int i = 0; i < 16; i++) {
            if (first + ks * 32 + (i >> 2) * 8 + hi * 4 + (i & 3) > last_key) sacc[i] = kMasked;
          }
        }
        // row maximum over this lane's 16 keys, then over the two lanes of the row
        const float a0 = max3(sacc[0], sacc[1], sacc[2]), a1 = max3(sacc[3], sacc[4], sacc[5]);
        const float a2 = max3(sacc[6], sacc[7], sacc[8]), a3 = max3(sacc[9], sacc[10], sacc[11]);
        const float a4 = max3(sacc[12], sacc[13], sacc[14]);
        const float mn = max_across_halves(max3(max3(a0, a1, a2), max3(a3, a4, sacc[15]), m));
        // The reference m only has to keep the exponentials in range, so it follows the maximum lazily: sums
        // and outputs move to a new reference only when some row's maximum exceeds the current one by more than
        // 2^kLazyBits in weight (weights then stay below that factor; fp32 sums and bf16 weights keep their
        // relative precision).  Without the slack ~60 % of the 32-key steps of a 4096-key context rescale.
        if (__any(mn > m + lazy)) {
          const float corr = ex2((m - mn) * c2);
          l *= corr;
#pragma unroll
          for (int d = 0; d < DB; d++)
#pragma unroll
            for (int i = 0; i < 16; i++) o[d][i] *= corr;
          m = mn;
        }
        const float nmc = -m * c2;
        float e[16];
#pragma unroll
        for (int i = 0; i < 16; i++) e[i] = ex2(fmaf(sacc[i], c2, nmc));
        l += ((e[0] + e[1]) + (e[2] + e[3])) + ((e[4] + e[5]) + (e[6] + e[7])) +
             (((e[8] + e[9]) + (e[10] + e[11])) + ((e[12] + e[13]) + (e[14] + e[15])));
        // values 0..7 are the keys of the first 16-key step, 8..15 of the second
#pragma unroll
        for (int st = 0; st < 2; st++) {
          bf16x8 pf[PARTS];
          weight_frags<PARTS>(pf, e + 8 * st);
          if constexpr (CAREFUL) {
            const int key = first + ks * 32 + 16 * st + hi * 4;  // keys key + 0 .. 3, key + 8 .. 11
#pragma unroll
            for (int d = 0; d < DB; d++) {
              fence_sched();
              bf16x8 vd = read_vt_frag<HD>(vtile, ks, st, d, lane);
              add_not_finite(o[d], vd, key, last_key, e + 8 * st);
#pragma unroll
              for (int part = PARTS - 1; part >= 0; part--)
                o[d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vd, pf[part], o[d], 0, 0, 0);
            }
            fence_sched();
            continue;
          }
#pragma unroll
          for (int part = PARTS - 1; part >= 0; part--)
#pragma unroll
            for (int d = 0; d < DB; d++)  // DB independent accumulators back to back
              o[d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[d][st], pf[part], o[d], 0, 0, 0);
        }
      }
    }
    tile_ready();
  };
  auto all_keys = [&](auto careful) {
#pragma unroll
    for (int d = 0; d < DB; d++)
#pragma unroll
      for (int i = 0; i < 16; i++) o[d][i] = 0.f;
    m = kNoMax, l = 0.f;
    stage(0, first_tile + group);
    tile_ready();
    if (decltype(careful)::value) {
      for (int i = 0; i < steps; i++) tile_step(i & 1, careful, i);
      return;
    }
    for (int i = 0; i < steps; i += 2) {
      tile_step(std::integral_constant<int, 0>{}, careful, i);
      if (i + 1 < steps) tile_step(std::integral_constant<int, 1>{}, careful, i + 1);
    }
  };
  all_keys(std::false_type{});
  {
    float probe = l * 0.f;  // 0, or NaN where the lane's sums are not finite
#pragma unroll
    for (int d = 0; d < DB; d++)
#pragma unroll
      for (int i = 0; i < 16; i++) probe = fmaf(o[d][i], 0.f, probe);
    const bool finite = !active || __all(probe == 0.f);
    int* waves = reinterpret_cast<int*>(smem);
    __syncthreads();  // the tiles have been read
    if (lane == 0) waves[wave] = finite;
    __syncthreads();
    const bool all_finite = __all(waves[lane % (RW * KW)] != 0);
    __syncthreads();  // the tiles' place is free again
    if (!all_finite) all_keys(std::true_type{});
  }

  if constexpr (KW > 1) {
    // merge the key groups' (m, l, O), half of them into the other half at a time, through the tiles' LDS
    constexpr int kRegion = (DB * 16 + 4) * 64 * 4;  // one wave's: DB x 4 float4 and one float2 (padded) per lane
    static_assert(KW / 2 * RW * kRegion <= KW * (int)attention_group_lds<HD, TK>(), "merge regions");
#pragma unroll
    for (int s = KW / 2; s >= 1; s >>= 1) {
      __syncthreads();
      float4* region = reinterpret_cast<float4*>(smem + ((group & (s - 1)) * RW + rwave) * kRegion) + lane;
      if (group >= s && group < 2 * s) {
#pragma unroll
        for (int d = 0; d < DB; d++)
#pragma unroll
          for (int g = 0; g < 4; g++)
            region[(d * 4 + g) * 64] = make_float4(o[d][4 * g], o[d][4 * g + 1], o[d][4 * g + 2], o[d][4 * g + 3]);
        region[DB * 4 * 64] = make_float4(m, l, 0.f, 0.f);
      }
      __syncthreads();
      if (group < s) {
        const float4 ml = region[DB * 4 * 64];
        const float mn = fmaxf(m, ml.x);
        const float a = ex2((m - mn) * c2), c = ex2((ml.x - mn) * c2);
        m = mn, l = l * a + ml.y * c;
#pragma unroll
        for (int d = 0; d < DB; d++)
#pragma unroll
          for (int g = 0; g < 4; g++) {
            const float4 x = region[(d * 4 + g) * 64];
            o[d][4 * g] = o[d][4 * g] * a + x.x * c, o[d][4 * g + 1] = o[d][4 * g + 1] * a + x.y * c;
            o[d][4 * g + 2] = o[d][4 * g + 2] * a + x.z * c, o[d][4 * g + 3] = o[d][4 * g + 3] * a + x.w * c;
          }
      }
    }
  }
  if (!active || group != 0) return;
  const float l_row = l + __shfl_xor(l, 32);
  if (key_splits > 1) {  // as it is, for merge_attention
    if (row_ok) {
      const size_t rec = (size_t)unit * pl.R + r, all = (size_t)pl.nb * pl.Hkv * key_splits * pl.R;
      if (hi == 0) reinterpret_cast<float2*>(records + all * pl.d)[rec] = make_float2(m, l_row);
#pragma unroll
      for (int d = 0; d < DB; d++)
#pragma unroll
        for (int g = 0; g < 4; g++) {
          const int col = d * 32 + g * 8 + hi * 4;
          if (col < pl.d)
            *reinterpret_cast<float4*>(records + rec * pl.d + col) =
                make_float4(o[d][4 * g], o[d][4 * g + 1], o[d][4 * g + 2], o[d][4 * g + 3]);
        }
    }
    return;
  }
  const float inv = 1.0f / l_row;
  if (row_ok) {
    if (hi == 0) lse_out[orow] = (m * c2 + __log2f(l_row)) * 0.69314718055994530942f;
    bf16_t* dst = out + orow * pl.d;
#pragma unroll
    for (int d = 0; d < DB; d++) {
#pragma unroll
      for (int g = 0; g < 4; g++) {
        const int col = d * 32 + g * 8 + hi * 4;
        const f32x2 p0 = {o[d][4 * g + 0] * inv, o[d][4 * g + 1] * inv};
        const f32x2 p1 = {o[d][4 * g + 2] * inv, o[d][4 * g + 3] * inv};
        uint2 w;
        w.x = __builtin_bit_cast(unsigned int, __builtin_convertvector(p0, bf16x2));
        w.y = __builtin_bit_cast(unsigned int, __builtin_convertvector(p1, bf16x2));
        if (col < pl.d) *reinterpret_cast<uint2*>(dst + col) = w;
      }
    }
  }
}

// Output and normaliser of every row from its key splits: LANES threads per row, four columns each; eight splits are loaded together.
template <int LANES>
__global__ __launch_bounds__(256) void merge_attention(const float* __restrict__ records, bf16_t* __restrict__ out,
                                                       float* __restrict__ lse_out, int key_splits, Plan pl) {
  constexpr int kAtOnce = 8;
  const int64_t row = (int64_t)blockIdx.x * (256 / LANES) + threadIdx.x / LANES, rows = (int64_t)pl.nb * pl.Hkv * pl.R;
  const int col = threadIdx.x % LANES * 4;
  if (row >= rows || col >= pl.d) return;
  const int bh = (int)(row / pl.R), r = (int)(row - (int64_t)bh * pl.R);
  const float2* sums = reinterpret_cast<const float2*>(records + rows * key_splits * pl.d);
  float m = kNoMax, l = 0.f, o[4] = {0.f, 0.f, 0.f, 0.f};
  for (int s0 = 0; s0 < key_splits; s0 += kAtOnce) {
    float2 ml[kAtOnce];
    float4 x[kAtOnce];
#pragma unroll
    for (int i = 0; i < kAtOnce; i++) {
      const size_t rec = ((size_t)bh * key_splits + min(s0 + i, key_splits - 1)) * pl.R + r;
      ml[i] = sums[rec];
      x[i] = *reinterpret_cast<const float4*>(records + rec * pl.d + col);
    }
    float mn = m;
#pragma unroll
    for (int i = 0; i < kAtOnce; i++) mn = fmaxf(mn, ml[i].x);
    const float old = ex2((m - mn) * pl.c2);
    l *= old;
#pragma unroll
    for (int j = 0; j < 4; j++) o[j] *= old;
    m = mn;
#pragma unroll
    for (int i = 0; i < kAtOnce; i++) {
      if (s0 + i >= key_splits) break;
      const float a = ex2((ml[i].x - mn) * pl.c2);
      l = fmaf(ml[i].y, a, l);
      o[0] = fmaf(x[i].x, a, o[0]), o[1] = fmaf(x[i].y, a, o[1]), o[2] = fmaf(x[i].z, a, o[2]), o[3] = fmaf(x[i].w, a, o[3]);
    }
  }
  const float inv = 1.0f / l;
  const f32x2 p0 = {o[0] * inv, o[1] * inv}, p1 = {o[2] * inv, o[3] * inv};
  uint2 w;
  w.x = __builtin_bit_cast(unsigned int, __builtin_convertvector(p0, bf16x2));
  w.y = __builtin_bit_cast(unsigned int, __builtin_convertvector(p1, bf16x2));
  // rows of a head are G query heads of p tokens each: dense in `out`
  *reinterpret_cast<uint2*>(out + row * pl.d + col) = w;
  if (col == 0) lse_out[row] = (m * pl.c2 + __log2f(l)) * 0.69314718055994530942f;
}

// ---------------------------------------------------------------------------------------- plain fp32 form
__device__ __forceinline__ float to_f32(float x) { return x; }
__device__ __forceinline__ float to_f32(__hip_bfloat16 x) { return __bfloat162float(x); }
__device__ __forceinline__ void from_f32(float& dst, float x) { dst = x; }
__device__ __forceinline__ void from_f32(__hip_bfloat16& dst, float x) { dst = __float2bfloat16(x); }

// One workgroup per query row.  Keys are taken 256 at a time: thread i scores key i, the chunk's maximum
// and sum update the running pair, then thread c accumulates head_dim column c over the chunk's keys.
template <typename T>
__global__ __launch_bounds__(256) void patch_attention_plain(const T* __restrict__ q, const T* __restrict__ k,
                                                             const T* __restrict__ v, T* __restrict__ out,
                                                             float* __restrict__ lse_out, Plan pl) {
  __shared__ float qs[256], w[256], red[4];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int t = blockIdx.x % pl.p, hq = (blockIdx.x / pl.p) % pl.Hq, b = blockIdx.x / (pl.p * pl.Hq);
  const int h = hq / pl.G;
  const T* qrow = q + b * pl.qsb + (int64_t)hq * pl.qsh + (int64_t)t * pl.qst;
  for (int c = tid; c < pl.d; c += 256) qs[c] = to_f32(qrow[c]);
  __syncthreads();
  const T* kbase = k + b * pl.ksb + (int64_t)h * pl.ksh;
  const T* vbase = v + b * pl.ksb + (int64_t)h * pl.ksh;
  const int n_keys = ctx_rows(pl, b * pl.Hkv + h) + (pl.causal_patch ? t + 1 : 0);
  float m = -INFINITY, l = 0.f, acc = 0.f;  // acc: column tid of the output, relative to the reference m
  auto block_reduce = [&](float x, bool is_max) {
    for (int off = 32; off >= 1; off >>= 1) {
      const float o = __shfl_xor(x, off);
      x = is_max ? fmaxf(x, o) : x + o;
    }
    __syncthreads();  // red[] of the previous reduction has been read by everyone
    if (lane == 0) red[wave] = x;
    __syncthreads();
    return is_max ? fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3])) : (red[0] + red[1]) + (red[2] + red[3]);
  };
  for (int k0 = 0; k0 < n_keys; k0 += 256) {
    const int i = k0 + tid;
    float z = -INFINITY;
    if (i < n_keys) {
      const T* krow = kbase + (int64_t)i * pl.kst;
      float dot = 0.f;
      for (int c = 0; c < pl.d; c++) dot = fmaf(qs[c], to_f32(krow[c]), dot);
      z = dot * pl.c2;
    }
    const float mn = fmaxf(m, block_reduce(z, true));
    // a logit of -inf has weight 0, also while there has been no other: no -inf - -inf
    const float e = z == -INFINITY ? 0.f : exp2f(z - mn);
    const float corr = m == mn ? 1.f : exp2f(m - mn);  // first chunk: exp2(-inf) = 0 times 0
    const float s = block_reduce(e, false);
    l = l * corr + s;
    acc *= corr;
    m = mn;
    w[tid] = e;
    __syncthreads();
    if (tid < pl.d) {
      const int cnt = min(256, n_keys - k0);
      for (int j = 0; j < cnt; j++) acc = fmaf(w[j], to_f32(vbase[(int64_t)(k0 + j) * pl.kst + tid]), acc);
    }
    __syncthreads();  // w[] is rewritten by the next chunk
  }
  const size_t orow = ((size_t)b * pl.Hq + hq) * pl.p + t;
  if (tid < pl.d) from_f32(out[orow * pl.d + tid], n_keys > 0 ? acc / l : 0.f);  // no key at all: O = 0, lse = -inf
  if (tid == 0) lse_out[orow] = n_keys > 0 ? (m + log2f(l)) * 0.69314718055994530942f : -INFINITY;
}

template <int HD, int KS, int DB, int PARTS, int RW, int KW, int TK>
hipError_t launch_one(const Plan& pl, const AttentionShape& shape, const void* q, const void* k, const void* v, void* out,
                      float* lse, float* room, hipStream_t stream) {
  const auto kernel = patch_attention_mfma<HD, KS, DB, PARTS, RW, KW, TK>;
  const int n_rb = (pl.R + 32 * RW - 1) / (32 * RW);
  const size_t smem = KW * attention_group_lds<HD, TK>();
  if (smem > 64 * 1024) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)smem);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(kernel, dim3(8 * n_rb, (pl.nb * pl.Hkv * shape.key_splits + 7) / 8), dim3(RW * KW * 64), smem, stream,
                     static_cast<const bf16_t*>(q), static_cast<const bf16_t*>(k), static_cast<const bf16_t*>(v),
                     static_cast<bf16_t*>(out), lse, room, shape.key_splits, shape.split_keys, pl);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess || shape.key_splits == 1) return e;
  constexpr int kLanes = DB * 8;
  constexpr int kPerRow = kLanes == 24 ? 32 : kLanes;
  const int64_t rows = (int64_t)pl.nb * pl.Hkv * pl.R;
  hipLaunchKernelGGL(merge_attention<kPerRow>, dim3((unsigned)((rows + 256 / kPerRow - 1) / (256 / kPerRow))), dim3(256), 0,
                     stream, room, static_cast<bf16_t*>(out), lse, shape.key_splits, pl);
  return hipGetLastError();
}

template <int HD, int KS, int DB, int PARTS>
hipError_t launch_mfma(const Plan& pl, const void* q, const void* k, const void* v, void* out, float* lse, float* room,
                       hipStream_t stream) {
  constexpr int kMostGroups = HD == 64 ? 8 : 4;
  const AttentionShape shape = attention_shape(pl, room != nullptr);
  if (shape.row_waves == 8) return launch_one<HD, KS, DB, PARTS, 8, 1, 64>(pl, shape, q, k, v, out, lse, room, stream);
  if (shape.row_waves == 4) return launch_one<HD, KS, DB, PARTS, 4, 2, 64>(pl, shape, q, k, v, out, lse, room, stream);
  if (shape.row_waves == 2) return launch_one<HD, KS, DB, PARTS, 2, 4, 32>(pl, shape, q, k, v, out, lse, room, stream);
  return launch_one<HD, KS, DB, PARTS, 1, kMostGroups, 32>(pl, shape, q, k, v, out, lse, room, stream);
}

}  // namespace

hipError_t launch_patch_attention(const Plan& pl, const void* q, const void* k, const void* v, void* out,
                                  float* lse, float* room_opt, hipStream_t stream) {
  if (pl.dtype == EPICACHE_DTYPE_BF16) {
    if (pl.d == 128) return launch_mfma<128, 8, 4, 1>(pl, q, k, v, out, lse, room_opt, stream);
    if (pl.d <= 32) return launch_mfma<64, 2, 1, 3>(pl, q, k, v, out, lse, room_opt, stream);
    if (pl.d <= 64) return launch_mfma<64, 4, 2, 3>(pl, q, k, v, out, lse, room_opt, stream);
    if (pl.d <= 96) return launch_mfma<128, 6, 3, 3>(pl, q, k, v, out, lse, room_opt, stream);
    if (pl.d < 128) return launch_mfma<128, 8, 4, 3>(pl, q, k, v, out, lse, room_opt, stream);
  }
  const unsigned rows = (unsigned)((size_t)pl.nb * pl.Hq * pl.p);
  if (pl.dtype == EPICACHE_DTYPE_F32)
    hipLaunchKernelGGL(patch_attention_plain<float>, dim3(rows), dim3(256), 0, stream, static_cast<const float*>(q),
                       static_cast<const float*>(k), static_cast<const float*>(v), static_cast<float*>(out), lse, pl);
  else
    hipLaunchKernelGGL(patch_attention_plain<__hip_bfloat16>, dim3(rows), dim3(256), 0, stream,
                       static_cast<const __hip_bfloat16*>(q), static_cast<const __hip_bfloat16*>(k),
                       static_cast<const __hip_bfloat16*>(v), static_cast<__hip_bfloat16*>(out), lse, pl);
  return hipGetLastError();
}

}  // namespace epicache

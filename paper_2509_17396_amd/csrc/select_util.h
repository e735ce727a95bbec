// Device helpers shared by the selection kernels (uniform top-M and ragged / pooled selection).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace epicache {

// Unsigned key whose integer order is the IEEE-754 total order of the float.
__device__ __forceinline__ uint32_t order_key(float x) {
  const uint32_t u = __float_as_uint(x);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

__device__ __forceinline__ int lanes_below(uint64_t mask) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                   __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0));
}

// Sum, minimum and maximum over the first LANES lanes of every group of LANES consecutive lanes (4, 8 or 16), in all
// of them, with lane permutations inside a 16-lane row: (i, i^1), (i, i^2), i <-> 7-i, i <-> 15-i.
template <int LANES, typename Op>
__device__ __forceinline__ uint32_t lanes_reduce(uint32_t x, Op op) {
  auto perm = [](uint32_t v, auto ctrl) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, decltype(ctrl)::value, 0xf, 0xf, false);
  };
  if (LANES >= 2) x = op(x, perm(x, std::integral_constant<int, 0xB1>{}));    // quad_perm [1,0,3,2]
  if (LANES >= 4) x = op(x, perm(x, std::integral_constant<int, 0x4E>{}));    // quad_perm [2,3,0,1]
  if (LANES >= 8) x = op(x, perm(x, std::integral_constant<int, 0x141>{}));   // row_half_mirror
  if (LANES >= 16) x = op(x, perm(x, std::integral_constant<int, 0x140>{}));  // row_mirror
  return x;
}
// the same over the whole wave; the result is wave-uniform
template <typename Op>
__device__ __forceinline__ uint32_t wave_reduce(uint32_t x, Op op) {
  x = lanes_reduce<16>(x, op);
  const uint32_t a = __builtin_amdgcn_readlane(x, 0), b = __builtin_amdgcn_readlane(x, 16);
  const uint32_t c = __builtin_amdgcn_readlane(x, 32), d = __builtin_amdgcn_readlane(x, 48);
  return op(op(a, b), op(c, d));
}

// Inclusive sum over lanes 0 .. l of the wave.
__device__ __forceinline__ uint32_t wave_prefix(uint32_t x) {
  auto from = [](uint32_t v, auto ctrl, auto rows) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, decltype(ctrl)::value, decltype(rows)::value, 0xf, false);
  };
  constexpr std::integral_constant<int, 0xf> all;
  x += from(x, std::integral_constant<int, 0x111>{}, all);  // row_shr 1, 2, 4, 8: inside a row of 16 lanes
  x += from(x, std::integral_constant<int, 0x112>{}, all);
  x += from(x, std::integral_constant<int, 0x114>{}, all);
  x += from(x, std::integral_constant<int, 0x118>{}, all);
  x += from(x, std::integral_constant<int, 0x142>{}, std::integral_constant<int, 0xa>{});  // lane 15 of a row to the next one
  x += from(x, std::integral_constant<int, 0x143>{}, std::integral_constant<int, 0xc>{});  // lane 31 to the upper half
  return x;
}

// ---- Selection of the K largest of up to NW * 64 * VPT keys that a workgroup of NW waves holds in registers.
//
// Thread (wave, lane) holds keys of the indices base + 64 j, base = wave * 64 * VPT + lane, j < VPT, as order_key()
// values; indices at or beyond n hold 0.  The interval [lo, hi] that must contain the K-th largest key starts at the
// row's own minimum and maximum and is cut into up to 1024 equal parts, whose keys are counted in LDS; the part that holds the
// K-th key is the next interval.  Keys in [lo, hi] of which there are at most 64 are ranked against each other, in every
// wave for itself.  Equal parts of the range that the scores cover hold few keys each, so one cut is nearly always
// enough.  The lowest part's count follows from the others': keys there (most of a row where weights have underflowed to 0) are
// not counted, and the filler behind a row never is.  Other parts may be crowded as well (a tight cluster and a few scores
// far from it), and LDS takes the keys of one part one after the other: a wave of whose second 64 keys many meet, by a
// look at neighbouring lanes, counts that part in a register.  (8 rows of 24576, a hundred values and 1 % of outliers: 56.3 us
// counted one by one, 20.8 so; smooth rows take 12.4 instead of 12.3.  Waves of 256 keys have no more than 4 meetings; the look
// would take a fused small step 0.2 us.)
// Bound by its chain of dependent steps: reduce the range, count, find the part, gather, rank, a barrier between each.  It
// replaces cuts into four by counting the keys at or above three values, a barrier each, six to ten of them: 32 rows of 512
// scores 6.5 -> 4.3 us, of 4096 9.5 -> 5.7, of 8192 11.4 -> 8.4; 896 rows of 4096 16.8 -> 12.3; 256 rows of 24576 26.6 -> 20.5.
constexpr int kCandidates = 64;
constexpr int kParts = 1024;
constexpr int kCrowd = 16;  // of 64 lanes: half the keys in one part leave 16 pairs

template <int NW>
struct SelectLds {
  __attribute__((aligned(16))) uint32_t parts[kParts];
  __attribute__((aligned(16))) uint32_t cand[kCandidates];
  uint32_t n_cand;
  uint2 range[NW];
  uint2 before[NW];
};

// emit_kept's `put`: into out[0, cap)
struct IntoRow {
  int32_t* __restrict__ out;
  uint32_t cap;
  __device__ __forceinline__ void operator()(uint32_t place, int index) const {
    if (place < cap) out[place] = index;
  }
};

struct Threshold {
  uint32_t thr;      // the K-th largest key
  uint32_t need_eq;  // how many keys equal to it are kept (the first ones in index order), >= 1
  bool cut;          // some keys equal to it are not kept
};

// count += key >= t for four keys.  By hand because the comparisons fill the two wait states that gfx950 wants between a
// comparison and the add that takes its mask as the carry; the compiler puts idle cycles there instead.
__device__ __forceinline__ void count4(uint32_t& count, const uint32_t* key, uint32_t t) {
  uint64_t m0, m1, m2, m3;
  asm("v_cmp_le_u32_e64 %1, %5, %6\n\t"
      "v_cmp_le_u32_e64 %2, %5, %7\n\t"
      "v_cmp_le_u32_e64 %3, %5, %8\n\t"
      "v_cmp_le_u32_e64 %4, %5, %9\n\t"
      "v_addc_co_u32_e64 %0, %1, 0, %0, %1\n\t"
      "v_addc_co_u32_e64 %0, %2, 0, %0, %2\n\t"
      "v_addc_co_u32_e64 %0, %3, 0, %0, %3\n\t"
      "v_addc_co_u32_e64 %0, %4, 0, %0, %4"
      : "+v"(count), "=&s"(m0), "=&s"(m1), "=&s"(m2), "=&s"(m3)
      : "s"(t), "v"(key[0]), "v"(key[1]), "v"(key[2]), "v"(key[3]));
}

// Keeps the masks of one group of 64 keys from being computed ahead for all groups, which spills scalar registers.
__device__ __forceinline__ void one_group_at_a_time() { __builtin_amdgcn_sched_barrier(0); }

// f(j) for the groups of 64 keys that the waves hold: all VPT, or (PARTIAL) the first `groups` of them, a multiple of
// kGroupsAtOnce, where the rows turn out shorter than the kernel has registers for.
constexpr int kGroupsAtOnce = 4;
template <int VPT, bool PARTIAL, typename F>
__device__ __forceinline__ void each_group(int groups, F f) {
#pragma unroll
  for (int j0 = 0; j0 < VPT; j0 += kGroupsAtOnce) {
    if (PARTIAL && j0 >= groups) continue;
#pragma unroll
    for (int j = j0; j < j0 + kGroupsAtOnce; j++) f(j);
  }
}

// x of lane ^ 1
__device__ __forceinline__ uint32_t lane_beside(uint32_t x) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0xB1, 0xf, 0xf, false);
}

// The loads are unconditional (indices behind the row re-read its last score): behind a branch each would wait for the
// one before it.
template <int VPT, bool PARTIAL = false>
__device__ __forceinline__ void load_keys(uint32_t (&keys)[VPT], uint32_t& least, const float* __restrict__ row,
                                          int base, int n, int groups = VPT) {
  float x[VPT];
  least = 0xffffffffu;
  if (__builtin_amdgcn_readfirstlane(base) + groups * 64 <= n) {  // the wave's indices all lie inside the row
    each_group<VPT, PARTIAL>(groups, [&](int j) { x[j] = row[base + j * 64]; });
    each_group<VPT, PARTIAL>(groups, [&](int j) {
      keys[j] = order_key(x[j]);
      least = min(least, keys[j]);
    });
    return;
  }
  each_group<VPT, PARTIAL>(groups, [&](int j) { x[j] = row[max(min(base + j * 64, n - 1), 0)]; });
  each_group<VPT, PARTIAL>(groups, [&](int j) {
    const uint32_t key = order_key(x[j]);
    least = min(least, key);  // of the row's own keys, not of the filler behind them
    keys[j] = base + j * 64 < n ? key : 0u;
  });
  if (n <= 0) least = 0xffffffffu;
}

// 1 <= K < n.  Called by all threads of the workgroup; every thread gets the same answer.  `least`: the smallest key
// of the thread.  Where 0 is a key of the row as well as the filler behind it, the missing candidates are zeros.
template <int VPT, int NW, bool PARTIAL = false>
__device__ __forceinline__ Threshold select_threshold(const uint32_t (&keys)[VPT], uint32_t least, int n, uint32_t K,
                                                      int wave, int lane, SelectLds<NW>& sm, int groups = VPT) {
  auto add = [](uint32_t a, uint32_t b) { return a + b; };
  auto lower = [](uint32_t a, uint32_t b) { return a < b ? a : b; };
  auto higher = [](uint32_t a, uint32_t b) { return a > b ? a : b; };
  auto clear_parts = [&] {
    for (int i = wave * 64 + lane; i < kParts / 4; i += NW * 64) reinterpret_cast<uint4*>(sm.parts)[i] = make_uint4(0, 0, 0, 0);
  };
  clear_parts();
  if (wave == 0) {
    sm.cand[lane] = 0;
    if (lane == 0) sm.n_cand = 0;
  }
  uint32_t mx = 0;
  each_group<VPT, PARTIAL>(groups, [&](int j) { mx = higher(mx, keys[j]); });
  const uint32_t mn = wave_reduce(least, lower);
  mx = wave_reduce(mx, higher);
  if (lane == 0) sm.range[wave] = make_uint2(mn, mx);
  __syncthreads();
  const uint2 r = sm.range[lane & (NW - 1)];
  // the K-th largest key lies in [lo, hi]: at_least_lo >= K > above_hi
  uint32_t lo = __builtin_amdgcn_readfirstlane(lanes_reduce<NW>(r.x, lower));
  uint32_t hi = __builtin_amdgcn_readfirstlane(lanes_reduce<NW>(r.y, higher));
  uint32_t at_least_lo = (uint32_t)n, above_hi = 0;
  bool again = false;
  while (lo < hi && at_least_lo - above_hi > kCandidates) {
    if (again) {
      __syncthreads();  // every wave has read the counts
      clear_parts();
      __syncthreads();
    }
    again = true;
    const uint32_t w = hi - lo;
    const int shift = max(0, 22 - __clz((int)w));  // w >> shift < kParts
    const uint32_t sample = (keys[1] - lo) >> shift;
    const uint64_t pairs = VPT <= 4 ? 0 : __ballot(sample == lane_beside(sample) && sample != 0 && keys[1] - lo <= w);
    if (__popcll(pairs) < kCrowd) {
      each_group<VPT, PARTIAL>(groups, [&](int j) {
        one_group_at_a_time();
        const uint32_t d = keys[j] - lo, part = d >> shift;
        if (d <= w && part != 0) atomicAdd(&sm.parts[part], 1u);
      });
    } else {
      const uint32_t crowd = __builtin_amdgcn_readlane(sample, __ffsll((unsigned long long)pairs) - 1);
      uint32_t there = 0;
      each_group<VPT, PARTIAL>(groups, [&](int j) {
        one_group_at_a_time();
        const uint32_t d = keys[j] - lo, part = d >> shift;
        there += __popcll(__ballot(d <= w && part == crowd));
        if (d <= w && part != 0 && part != crowd) atomicAdd(&sm.parts[part], 1u);
      });
      if (lane == 0) atomicAdd(&sm.parts[crowd], there);
    }
    __syncthreads();
    // lane l has parts 16 (63 - l) .. 16 (63 - l) + 15, lane 0 the highest ones
    const uint4* mine = reinterpret_cast<const uint4*>(sm.parts) + (63 - lane) * 4;
    const uint4 a = mine[0], b = mine[1], c = mine[2], d = mine[3];
    const uint32_t sum = ((a.x + a.y) + (a.z + a.w)) + ((b.x + b.y) + (b.z + b.w)) +
                         (((c.x + c.y) + (c.z + c.w)) + ((d.x + d.y) + (d.z + d.w)));
    const uint32_t incl = wave_prefix(sum);
    const uint32_t want = K - above_hi;  // rank in [lo, hi]
    const uint64_t reach = __ballot(incl >= want);
    if (reach == 0) {  // not in the parts that were counted: in the lowest one
      above_hi += __builtin_amdgcn_readlane(incl, 63);
      hi = lo + ((1u << shift) - 1);
    } else {
      const int l = __ffsll((unsigned long long)reach) - 1;
      const uint32_t before = __builtin_amdgcn_readlane(incl - sum, l);  // keys in the parts of the lanes before
      const int top = 16 * (63 - l) + 15;
      const uint32_t count = sm.parts[top - (lane & 15)];
      const uint32_t upto = before + wave_prefix(lane < 16 ? count : 0u);
      const int i = __ffsll((unsigned long long)__ballot(upto >= want)) - 1;
      const uint32_t there = __builtin_amdgcn_readlane(upto, i), held = __builtin_amdgcn_readlane(count, i);
      lo += (uint32_t)(top - i) << shift;
      hi = lower(hi, lo + ((1u << shift) - 1));
      at_least_lo = above_hi + there;
      above_hi = at_least_lo - held;
    }
  }
  if (lo >= hi) {  // all keys of the interval are equal
    const uint32_t rank = K - above_hi;
    return Threshold{lo, rank, rank < at_least_lo - above_hi};
  }
  // at most 64 candidates, one per lane
  const uint32_t from = lo ? lo : 1u;
  uint32_t in_wave = 0;
  each_group<VPT, PARTIAL>(groups, [&](int j) { in_wave += keys[j] - from <= hi - from; });
  in_wave = wave_reduce(in_wave, add);
  if (in_wave) {
    uint32_t pos = 0;
    if (lane == 0) pos = atomicAdd(&sm.n_cand, in_wave);
    pos = __builtin_amdgcn_readfirstlane(pos);
    each_group<VPT, PARTIAL>(groups, [&](int j) {
      one_group_at_a_time();
      const bool in = keys[j] - from <= hi - from;
      const uint64_t mask = __ballot(in);
      const uint32_t slot_of = pos + lanes_below(mask);
      if (in && slot_of < kCandidates) sm.cand[slot_of] = keys[j];
      pos += __popcll(mask);
    });
  }
  __syncthreads();
  const uint32_t held = at_least_lo - above_hi, want = K - above_hi;
  const uint32_t mine = sm.cand[lane];
  uint32_t gt = 0, ge = 0;  // candidates above this lane's, and those and the ones equal to it
  for (uint32_t i = 0; i < (held + 3) / 4; i++) {
    const uint4 c = reinterpret_cast<const uint4*>(sm.cand)[i];
    gt += (c.x > mine) + (c.y > mine) + (c.z > mine) + (c.w > mine);
    ge += (c.x >= mine) + (c.y >= mine) + (c.z >= mine) + (c.w >= mine);
  }
  ge = lower(ge, held);  // the places behind the last candidate hold 0
  const uint64_t who = __ballot(lane < (int)held && gt < want && want <= ge);
  const int l = __ffsll((unsigned long long)who) - 1;
  const uint32_t above = __builtin_amdgcn_readlane(gt, l), upto = __builtin_amdgcn_readlane(ge, l);
  return Threshold{(uint32_t)__builtin_amdgcn_readlane(mine, l), want - above, want < upto};
}

// Hands the indices of the kept keys of this wave's row to put(place, index), places ascending with the index, and
// returns how many of that row's keys up to and including this wave's are kept.  The row is held by the waves first_wave ..
// of the workgroup; waves before that hold rows whose keys come first among ties.
template <int VPT, int NW, bool PARTIAL = false, typename Put>
__device__ __forceinline__ uint32_t emit_kept(const uint32_t (&keys)[VPT], int base, int n, const Threshold& t, Put put,
                                              int wave, int first_wave, int lane, SelectLds<NW>& sm, int groups = VPT) {
  auto add = [](uint32_t a, uint32_t b) { return a + b; };
  // Where every key equal to the threshold stays, one comparison decides.  (The filler behind a row equals a threshold
  // of 0 and takes the other path.)
  const bool plain = !t.cut && t.thr != 0;
  asm volatile("" : "+s"(n));  // the masks index < n are made here again, not carried from the loads in scalar registers
  uint32_t cgt = 0, ceq = 0;  // keys that stay whatever their order; ties of which only the first ones stay
  if (plain) {
#pragma unroll
    for (int j = 0; j < VPT; j += kGroupsAtOnce)
      if (!PARTIAL || j < groups) count4(cgt, keys + j, t.thr);
  } else {
    each_group<VPT, PARTIAL>(groups, [&](int j) {
      one_group_at_a_time();
      cgt += keys[j] > t.thr, ceq += keys[j] == t.thr && base + j * 64 < n;
    });
    ceq = wave_reduce(ceq, add);
  }
  cgt = wave_reduce(cgt, add);
  if (lane == 0) sm.before[wave] = make_uint2(cgt, ceq);
  __syncthreads();
  uint32_t gt_before = 0, eq_before = 0, eq_first = 0;
#pragma unroll
  for (int w = 0; w < NW; w++) {
    const uint2 c = sm.before[w];
    if (w < wave) eq_before += c.y;
    if (w < first_wave) eq_first += c.y;
    else if (w < wave) gt_before += c.x;
  }
  gt_before = __builtin_amdgcn_readfirstlane(gt_before);
  if (plain) {
    each_group<VPT, PARTIAL>(groups, [&](int j) {
      one_group_at_a_time();
      const bool is = keys[j] >= t.thr;
      const uint64_t mask = __ballot(is);
      const uint32_t pos = gt_before + lanes_below(mask);
      if (is) put(pos, base + j * 64);
      gt_before += __popcll(mask);
    });
    return gt_before;
  }
  eq_before = __builtin_amdgcn_readfirstlane(eq_before);
  const uint32_t eq_gone = min((uint32_t)__builtin_amdgcn_readfirstlane(eq_first), t.need_eq);  // kept in rows before
  each_group<VPT, PARTIAL>(groups, [&](int j) {
    one_group_at_a_time();
    const int i = base + j * 64;
    const bool is_gt = keys[j] > t.thr, is_eq = keys[j] == t.thr && i < n;
    const uint64_t bgt = __ballot(is_gt), beq = __ballot(is_eq);
    const uint32_t my_gt = gt_before + lanes_below(bgt), my_eq = eq_before + lanes_below(beq);
    if (is_gt || (is_eq && my_eq < t.need_eq)) {
      put(my_gt + min(my_eq, t.need_eq) - eq_gone, i);
    }
    gt_before += __popcll(bgt);
    eq_before += __popcll(beq);
  });
  return gt_before + min(eq_before, t.need_eq) - eq_gone;
}

// Histogram of one radix digit in LDS.  The scores of a row share few values of the leading digits (sign and
// exponent), so with a plain 256-bin array most of a wave's 64 atomics would meet on one address, which LDS
// serialises.  Every bin is therefore kept in kHistCopies copies, one per LDS bank (copy = lane % 32): at most two
// lanes of an instruction meet on an address.  hist_rep holds 256 * kHistCopies counters, all zero before a pass.
constexpr int kHistCopies = 32;

__device__ __forceinline__ void hist_count(uint32_t* hist_rep, uint32_t digit, int lane) {
  atomicAdd(&hist_rep[digit * kHistCopies + (lane & (kHistCopies - 1))], 1u);
}

// Between two workgroup barriers, by every thread of a workgroup of at least 256: thread t < 256 folds the copies
// of bin t into hist[t] (reading them in a rotated order, so the lanes of a wave stay on different banks) and
// clears them for the next pass.
__device__ __forceinline__ void hist_fold(uint32_t* hist_rep, uint32_t* hist, int tid) {
  if (tid < 256) {
    uint32_t sum = 0;
#pragma unroll 8
    for (int c = 0; c < kHistCopies; c++) {
      uint32_t& slot = hist_rep[tid * kHistCopies + ((c + tid) & (kHistCopies - 1))];
      sum += slot;
      slot = 0;
    }
    hist[tid] = sum;
  }
}

// One radix digit of a select: given the 256-bin histogram of the digit among the keys that still
// match the prefix, find the bin that holds the kth largest (kth >= 1 counts from the top) and how
// many keys lie in the bins above it.  Every wave calls this with the same arguments and gets the
// same answer; lane l owns bins 255-4l .. 252-4l.
__device__ __forceinline__ void locate_digit(const uint32_t* hist, uint32_t kth, int lane, uint32_t& bin,
                                             uint32_t& above) {
  uint32_t c[4];
#pragma unroll
  for (int x = 0; x < 4; x++) c[x] = hist[255 - 4 * lane - x];
  const uint32_t mine = c[0] + c[1] + c[2] + c[3];
  uint32_t incl = mine;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const uint32_t o = __shfl_up(incl, off);
    if (lane >= off) incl += o;
  }
  const uint32_t excl = incl - mine;
  const bool here = excl < kth && kth <= incl;  // true in exactly one lane
  uint32_t b = 0, a = 0;
  if (here) {
    uint32_t run = excl;
#pragma unroll
    for (int x = 0; x < 4; x++) {
      if (run < kth && kth <= run + c[x]) {
        b = 255 - 4 * lane - x;
        a = run;
      }
      run += c[x];
    }
  }
  const uint64_t who = __ballot(here);
  const int src = __ffsll((unsigned long long)who) - 1;
  bin = __shfl(b, src);
  above = __shfl(a, src);
}

}  // namespace epicache

// Selection and compaction in one launch with a patience and with claims of the caller's choice, and the compaction with claims,
// for the tests.  Not part of the library.
#include <string.h>

#include "../compact.hip"

// scores [nb, hkv, n], keep [nb, hkv, m], k and v bf16 [nb, hkv, n, d], claims [nb, hkv, *claims_per_head], all dense.
extern "C" __attribute__((visibility("default"))) int select_compact_with_patience(
    int nb, int hkv, int d, int n, int m, const float* scores, uint32_t* claims, int32_t* keep, void* k, void* v, int patience,
    int* done, void* hip_stream) {
  if (!scores || !claims || !keep || !k || !v || !done || nb < 1 || hkv < 1 || d % 8 != 0 || d < 8 || d > 256 || n < 2 ||
      n > 16384 || m < 1 || m >= n || patience < 0)
    return EPICACHE_ERR_INVALID_ARG;
  epicache::Plan pl;
  memset(&pl, 0, sizeof(pl));
  pl.nb = nb, pl.Hkv = hkv, pl.d = d, pl.elem = 2, pl.dtype = EPICACHE_DTYPE_BF16;
  pl.N = n, pl.M = m, pl.n_keep = m, pl.keep_stride = m;
  pl.heads_magic = (uint32_t)(((uint64_t(1) << 32) + hkv - 1) / hkv);
  pl.kst = d, pl.ksh = (int64_t)n * d, pl.ksb = pl.ksh * hkv;
  pl.claims = claims;
  bool took = false;
  const hipError_t e =
      epicache::launch_select_compact(pl, pl, scores, keep, 0, k, v, (hipStream_t)hip_stream, &took, patience);
  *done = took;
  return e == hipSuccess ? EPICACHE_OK : EPICACHE_ERR_DEVICE;
}

// launch_compact as a step calls it: claims [nb, hkv, *claims_per_head] are clear; returns the number of ranges, 0 for none.
extern "C" __attribute__((visibility("default"))) int compact_with_claims(int nb, int hkv, int d, int elem, int n, int m,
                                                                          const int32_t* keep, uint32_t* claims, void* k, void* v,
                                                                          void* hip_stream) {
  if (!claims || !keep || !k || !v || nb < 1 || hkv < 1 || d % 8 != 0 || d < 8 || d > 256 || (elem != 2 && elem != 4) || n < 2 ||
      m < 1 || m >= n || (int64_t)nb * hkv > 65535)
    return -1;
  epicache::Plan pl;
  memset(&pl, 0, sizeof(pl));
  pl.nb = nb, pl.Hkv = hkv, pl.d = d, pl.elem = elem, pl.dtype = elem == 2 ? EPICACHE_DTYPE_BF16 : EPICACHE_DTYPE_F32;
  pl.N = n, pl.M = m, pl.n_keep = m, pl.keep_stride = m;
  pl.heads_magic = (uint32_t)(((uint64_t(1) << 32) + hkv - 1) / hkv);
  pl.kst = d, pl.ksh = (int64_t)n * d, pl.ksb = pl.ksh * hkv;
  pl.claims = claims;
  if (epicache::launch_compact(pl, keep, k, v, false, (hipStream_t)hip_stream) != hipSuccess) return -1;
  return epicache::compact_ranges_of(2 * (int64_t)nb * hkv, m, m, d * elem, false).parts;
}

extern "C" __attribute__((visibility("default"))) int claims_per_head(int* pitch) {
  *pitch = epicache::kClaimPitch;
  return epicache::kClaimsPerHead;
}

// The KeyDiff scoring with a patience of the caller's choice (0: every workgroup of the one-pass form does without the
// others), for the tests.  Not part of the library.
#include <string.h>

#include "../score_keydiff.hip"

extern "C" __attribute__((visibility("default"))) int keydiff_with_patience(
    int dtype, int nb, int hkv, int d, int n, int64_t ksb, int64_t ksh, int64_t kst, const void* k,
    const int32_t* n_ctx_opt, float* scores, void* workspace, size_t workspace_bytes, int patience, void* hip_stream) {
  if (!k || !scores || !workspace || nb < 1 || hkv < 1 || d % 8 != 0 || d < 8 || d > 256 || n < 1 || patience < 0 ||
      kst < d || ksh < kst * (int64_t)n || (nb > 1 && ksb < ksh * (int64_t)hkv))
    return EPICACHE_ERR_INVALID_ARG;
  epicache::Plan pl;
  memset(&pl, 0, sizeof(pl));
  pl.nb = nb, pl.Hkv = hkv, pl.d = d, pl.N = n, pl.dtype = dtype;
  pl.elem = dtype == EPICACHE_DTYPE_F32 ? 4 : 2;
  pl.heads_magic = (uint32_t)(((uint64_t(1) << 32) + hkv - 1) / hkv);
  pl.ksb = ksb, pl.ksh = ksh, pl.kst = kst;
  pl.n_ctx = n_ctx_opt;
  if (workspace_bytes < epicache::keydiff_workspace_bytes(pl)) return EPICACHE_ERR_WORKSPACE_TOO_SMALL;
  const hipError_t e = epicache::launch_score_keydiff(pl, k, scores, workspace, (hipStream_t)hip_stream, patience);
  return e == hipSuccess ? EPICACHE_OK : EPICACHE_ERR_DEVICE;
}

"""Selection and compaction in one launch whose claims something else has written: a range that does not exist moves nothing,
and a workgroup that waits for a range that nobody takes gives up and leaves its rows as they are.  Every launch ends."""
import ctypes
import os

import pytest
import torch

from paper_2509_17396_amd import build

pytestmark = pytest.mark.gpu
DEV = "cuda"
LOOKS = 200


def load():
    so = os.path.join(os.path.dirname(build.LIB), "selftest", "libselect_compact_patience.so")
    if not os.path.exists(so):
        build.build_selftests()
    lib = ctypes.CDLL(so)
    vp, i32 = ctypes.c_void_p, ctypes.c_int
    lib.select_compact_with_patience.argtypes = [i32, i32, i32, i32, i32, vp, vp, vp, vp, vp, i32, ctypes.POINTER(i32), vp]
    lib.claims_per_head.argtypes = [ctypes.POINTER(i32)]
    return lib


# claims of the K of head 0 before the launch, as (ranges taken, ranges reported): as pass 2 leaves them, range 0 taken by
# nobody, all of them taken, a float in their place
BEFORE = {"clear": (0, 0), "first_range_gone": (1, 0), "all_gone": (32, 0), "overwritten": (0x3f800000, 0x3f800000),
          "negative": (0xbf800000 - (1 << 32), 0)}


@pytest.mark.parametrize("before", BEFORE)
@pytest.mark.parametrize("heads,n,m,d", [(2, 4096, 2048, 128), (3, 1024, 700, 128), (1, 16384, 9000, 256), (2, 8000, 7999, 24)])
def test_claims_that_something_else_wrote(heads, n, m, d, before):
    lib, pitch, done = load(), ctypes.c_int(0), ctypes.c_int(0)
    per_head = lib.claims_per_head(ctypes.byref(pitch))
    print(f"[gpu test] select_compact claims={before} heads={heads} N={n} M={m} d={d}", flush=True)
    g = torch.Generator(device=DEV).manual_seed(n + d)
    scores = torch.rand(heads, n, device=DEV, generator=g)
    k0, v0 = (torch.randn(heads, n, d, device=DEV, generator=g).to(torch.bfloat16) for _ in range(2))
    best = [torch.sort(s, descending=True, stable=True).indices[:m].sort().values for s in scores.cpu()]
    claims = torch.zeros(heads, per_head, dtype=torch.int32, device=DEV)
    claims[0, 0], claims[0, pitch.value] = BEFORE[before]
    k, v, keep = k0.clone(), v0.clone(), torch.full((heads, m), -1, dtype=torch.int32, device=DEV)
    st = lib.select_compact_with_patience(1, heads, d, n, m, scores.data_ptr(), claims.data_ptr(), keep.data_ptr(), k.data_ptr(),
                                          v.data_ptr(), 1 << 14 if before == "clear" else LOOKS, ctypes.byref(done),
                                          torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert st == 0 and done.value == 1
    bits = lambda t: t.view(torch.int16)
    for h in range(heads):
        want = best[h].to(DEV)
        moved = before == "clear" or h > 0
        assert torch.equal(bits(v[h, :m]), bits(v0[h, want])) and torch.equal(bits(v[h, m:]), bits(v0[h, m:]))
        assert torch.equal(bits(k[h, :m]), bits(k0[h, want] if moved else k0[h, :m]))
        assert torch.equal(bits(k[h, m:]), bits(k0[h, m:]))
        if moved:
            assert torch.equal(keep[h].long(), want)
        else:  # written by the K of the head, as far as its ranges were taken
            assert bool(((keep[h] == -1) | (keep[h].long() == want)).all())
            assert int(keep[h, 0]) == -1 and (before == "first_range_gone" or bool((keep[h] == -1).all()))

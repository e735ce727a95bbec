"""KeyDiff scoring in one pass: a workgroup that does not wait for the others of its head adds up their sums itself, in the
same order, so the scores are the same bits whether none, some or all of them give up."""
import ctypes
import os

import pytest
import torch

from paper_2509_17396_amd import binding as ep
from paper_2509_17396_amd import build

pytestmark = pytest.mark.gpu


def load():
    so = os.path.join(os.path.dirname(build.LIB), "selftest", "libkeydiff_patience.so")
    if not os.path.exists(so):
        build.build_selftests()
    lib = ctypes.CDLL(so)
    vp, i64, i32 = ctypes.c_void_p, ctypes.c_int64, ctypes.c_int
    lib.keydiff_with_patience.argtypes = [i32, i32, i32, i32, i32, i64, i64, i64, vp, vp, vp, vp, ctypes.c_size_t, i32, vp]
    return lib


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("bf16", 64), ("f32", 64), ("f32", 32)])
@pytest.mark.parametrize("nb,heads,n", [(2, 3, 1025), (33, 8, 513), (2, 4, 4096), (1, 2, 16384), (1, 1, 60), (3, 1, 24001)])
def test_giving_up_gives_the_same_bits(dtype, d, nb, heads, n):
    lib = load()
    t = torch.float32 if dtype == "f32" else torch.bfloat16
    g = torch.Generator(device="cuda").manual_seed(n + d)
    k = (torch.randn(nb, heads, n, d, device="cuda", generator=g) + 0.3).to(t)
    k[0, 0, n // 2, 1] = float("nan")     # NaN sums are sums like any other
    lengths = torch.randint(0, n + 1, (nb, heads), device="cuda", generator=g, dtype=torch.int32)
    q = torch.empty(nb, heads, 1, d, dtype=t, device="cuda")
    prm = ep.make_params(q, k, n_cached=0, n_block=n, budget=1)
    size = ep.epicache_workspace_size(prm)
    for n_ctx in (None, lengths):
        want = torch.full((nb, heads, n), -7.0, device="cuda")
        ep.epicache_score_keydiff(prm, k, want, torch.empty(size, dtype=torch.uint8, device="cuda"), n_ctx=n_ctx)
        for patience in (0, 1, 3, 1 << 14):
            print(f"[gpu test] keydiff patience={patience} {dtype} d={d} nb={nb} heads={heads} N={n} ragged={n_ctx is not None}",
                  flush=True)
            # what the workspace held before does not count
            ws = torch.full((size,), patience % 251, dtype=torch.uint8, device="cuda")
            got = torch.full_like(want, -7.0)
            st = lib.keydiff_with_patience(
                ep.DTYPE_F32 if dtype == "f32" else ep.DTYPE_BF16, nb, heads, d, n, *k.stride()[:3], k.data_ptr(),
                n_ctx.data_ptr() if n_ctx is not None else None, got.data_ptr(), ws.data_ptr(), size, patience,
                torch.cuda.current_stream().cuda_stream)
            assert st == ep.OK
            assert torch.equal(got.view(torch.int32), want.view(torch.int32)), patience

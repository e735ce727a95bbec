"""What the size queries report: the attention step's room for key splits is asked for by its callers only.  Host code only."""
import ctypes

import pytest

from paper_2509_17396_amd import binding as ep


def params(nb, hq, hkv, p, d, n, m, causal, dtype=ep.DTYPE_BF16):
    cap = n + (p if causal else 0)
    return ep.Params(ctypes.sizeof(ep.Params), nb, hq, hkv, d, m, n - m, m, p, dtype, ep.REDUCE_SUM, 0.0, causal, 0,
                     hq * p * d, p * d, d, hkv * cap * d, cap * d, d)


def size_of(query, prm):
    out = ctypes.c_size_t(0)
    assert query(ctypes.byref(prm), ctypes.byref(out)) == ep.OK
    return out.value


# items, query heads, KV heads, patch, head_dim, rows, budget, causal: bytes of any step, and of one in overlapped chunks: statistics of the
# rows (a pair per key split and one number more), scores, kept indices, normalisers
@pytest.mark.parametrize("sizes,step,chunks", [
    ((4, 24, 8, 64, 128, 4096, 2048, 0), 1228800, 1), ((3, 32, 8, 64, 128, 4337, 3000, 0), 1245184, 1),
    ((1, 8, 2, 128, 128, 18000, 16000, 1), 542464, 1), ((1, 4, 4, 32, 64, 12000, 6000, 1), 355072, 1),
    ((128, 32, 8, 128, 128, 8192, 4096, 0), 71303168, 16)])
def test_only_the_attention_step_is_given_room_for_key_splits(sizes, step, chunks):
    lib, prm = ep.load(), params(*sizes)
    assert size_of(lib.epicache_workspace_size, prm) == step
    assert ep.epicache_overlapped_workspace_size(prm, 0) == (step, chunks)
    room = size_of(lib.epicache_attn_workspace_size, prm) - step
    assert (room > 0) == (chunks == 1) and room % 256 == 0
    assert ep.epicache_workspace_size(prm) == step + room and ep.epicache_workspace_size(prm, attention=False) == step


def test_one_workspace_for_all_calls_has_the_room_unless_told_otherwise():
    prm = params(4, 24, 8, 64, 128, 4096, 2048, 0)
    assert ep.epicache_workspace_size(prm) > ep.epicache_workspace_size(prm, attention=False)
    assert ep.alloc_workspace(prm, device="cpu").numel() == ep.epicache_workspace_size(prm)
    assert ep.alloc_workspace(prm, device="cpu", attention=False).numel() == ep.epicache_workspace_size(prm, attention=False)


@pytest.mark.parametrize("d,dtype", [(136, ep.DTYPE_BF16), (256, ep.DTYPE_BF16), (64, ep.DTYPE_F32)])
def test_no_room_for_rows_that_are_never_split(d, dtype):
    lib, prm = ep.load(), params(1, 4, 4, 32, d, 12000, 6000, 1, dtype)
    assert size_of(lib.epicache_attn_workspace_size, prm) == size_of(lib.epicache_workspace_size, prm)


def test_attention_size_checks_its_arguments():
    lib, prm = ep.load(), params(1, 4, 4, 32, 64, 12000, 6000, 1)
    assert lib.epicache_attn_workspace_size(ctypes.byref(prm), None) == ep.ERR_INVALID_ARG
    assert lib.epicache_attn_workspace_size(None, ctypes.byref(ctypes.c_size_t())) == ep.ERR_INVALID_ARG
    prm.struct_size -= 4
    assert lib.epicache_attn_workspace_size(ctypes.byref(prm), ctypes.byref(ctypes.c_size_t())) == ep.ERR_INVALID_ARG

"""The library's own chunk count of the overlapped steps (n_chunks = 0), host code only: the number it reports, given back
as n_chunks, is the same cut with the same workspace, and types and row lengths that were never measured in chunks run as
the plain step."""
import ctypes

import pytest

from paper_2509_17396_amd import binding as ep


def dense_params(nb, hkv, g, p, d, n_cached, n_block, dtype):
    hq, cap = hkv * g, n_cached + n_block
    return ep.Params(ctypes.sizeof(ep.Params), nb, hq, hkv, d, n_cached, n_block, n_cached, p, dtype, ep.REDUCE_SUM, 0.0,
                     0, 0, hq * p * d, p * d, d, hkv * cap * d, cap * d, d)


def plan(prm, n_chunks, with_lse, select):
    size, cap, used = ctypes.c_size_t(0), ctypes.c_int32(0), ctypes.c_int32(0)
    lib, ref = ep.load(), ctypes.byref
    if select is None:
        st = lib.epicache_overlapped_workspace_size(ref(prm), n_chunks, with_lse, ref(size), ref(used))
    else:
        st = lib.epicache_ragged_overlapped_workspace_size(ref(prm), select, n_chunks, with_lse, ref(size), ref(cap), ref(used))
    assert st == ep.OK
    return size.value, used.value


@pytest.mark.parametrize("with_lse", [0, 1])
@pytest.mark.parametrize("select", [None, ep.SELECT_PER_HEAD, ep.SELECT_POOLED])
@pytest.mark.parametrize("nb,hkv", [(48, 8), (50, 8), (97, 4), (128, 8), (130, 8), (131, 8), (225, 4), (1000, 1), (511, 128)])
def test_the_reported_count_makes_the_same_chunks(nb, hkv, select, with_lse):
    prm = dense_params(nb, hkv, 4, 128, 128, 4096, 4096, ep.DTYPE_BF16)
    size, used = plan(prm, 0, with_lse, select)
    assert used > 1
    assert plan(prm, used, with_lse, select) == (size, used)


@pytest.mark.parametrize("dtype,d,chunks", [(ep.DTYPE_BF16, 128, 16), (ep.DTYPE_BF16, 64, 8), (ep.DTYPE_BF16, 96, 1),
                                            (ep.DTYPE_BF16, 256, 1), (ep.DTYPE_F32, 64, 1), (ep.DTYPE_F32, 128, 1)])
def test_only_measured_rows_are_cut(dtype, d, chunks):
    assert plan(dense_params(128, 8, 4, 128, d, 4096, 4096, dtype), 0, 0, None)[1] == chunks


@pytest.mark.parametrize("select,chunks", [(None, 14), (ep.SELECT_PER_HEAD, 14), (ep.SELECT_POOLED, 7)])
def test_pooled_selection_gets_chunks_of_twice_the_pairs(select, chunks):
    assert plan(dense_params(224, 4, 7, 64, 128, 6000, 3500, ep.DTYPE_BF16), 0, 0, select)[1] == chunks
    # not with fewer than three of them
    assert plan(dense_params(95, 4, 7, 64, 128, 6000, 3500, ep.DTYPE_BF16), 0, 0, select)[1] == 5

"""Which contexts are scored with one product per logit (csrc/launch_rules.h, row_splits), and the wait states of that kernel's
hand-written instructions.  Host code only."""
import ctypes
import os

import pytest

from paper_2509_17396_amd import binding as ep
from paper_2509_17396_amd import build
from tests import test_isa_hazards as hz

BF16, F32 = ep.DTYPE_BF16, ep.DTYPE_F32
PLENTY = 1 << 40


@pytest.fixture(scope="module")
def splits():
    so = os.path.join(os.path.dirname(build.LIB), "selftest", "liblaunch_rules.so")
    if not os.path.exists(so):
        build.build_selftests()
    fn = ctypes.CDLL(so).row_splits
    fn.argtypes = [ctypes.c_int] * 8 + [ctypes.c_longlong]
    return fn


# dtype, head_dim, heads, rows, keys
@pytest.mark.parametrize("blocks,sizes", [
    # 1.02 to 1.6 times as long as two passes
    (0, [(BF16, 128, 8, 64, 2048), (BF16, 128, 4, 32, 1536), (BF16, 128, 896, 64, 384), (BF16, 128, 896, 128, 1280),
         (BF16, 128, 64, 192, 900), (BF16, 96, 896, 96, 600), (BF16, 96, 4, 64, 2048), (BF16, 64, 896, 128, 384),
         (BF16, 64, 4, 32, 2048), (F32, 64, 8, 64, 600), (F32, 64, 64, 32, 1024), (F32, 64, 16, 64, 2048)]),
    # 0.56 to 0.98
    (1, [(BF16, 128, 8, 32, 768), (BF16, 128, 896, 32, 2048), (BF16, 64, 4, 20, 384), (F32, 64, 896, 32, 384)]),
    (2, [(BF16, 128, 896, 64, 2048), (BF16, 96, 64, 64, 2024), (BF16, 64, 1792, 64, 768), (F32, 64, 32, 64, 1024)]),
    (4, [(BF16, 128, 896, 128, 2048), (BF16, 128, 64, 128, 384), (F32, 64, 2, 128, 384), (F32, 64, 256, 128, 1280)]),
    (8, [(BF16, 128, 32, 256, 2048), (BF16, 64, 64, 256, 900), (F32, 64, 128, 256, 2048)])])
def test_goes_where_it_is_faster(splits, blocks, sizes):
    for dtype, d, heads, rows, n in sizes:
        assert splits(dtype, d, heads, rows, rows, n, 0, 0, PLENTY) == blocks, (dtype, d, heads, rows, n)


def test_what_the_kernel_is_not_made_for(splits):
    for n, patch, causal, taken in [(2048, 32, 0, 1), (2049, 32, 0, 0), (2016, 32, 1, 1), (2017, 32, 1, 0)]:
        assert splits(BF16, 128, 512, 32, patch, n, causal, 0, PLENTY) == taken, n
    assert splits(BF16, 128, 512, 32, 32, 2048, 0, 1, PLENTY) == 0    # lengths of their own
    assert splits(F32, 64, 512, 257, 257, 2048, 0, 0, PLENTY) == 0    # nine blocks of rows
    for dtype, dims in ((BF16, (64, 72, 80, 88, 96, 128)), (F32, (64,))):
        for d in range(8, 257, 8):
            assert (splits(dtype, d, 64, 64, 64, 400, 0, 0, PLENTY) > 0) == (d in dims), (dtype, d)


@pytest.mark.parametrize("dtype,d", [(BF16, 64), (BF16, 80), (BF16, 128), (F32, 64)])
def test_parts_fit_their_room(splits, dtype, d):
    """Never more than the room holds, and at most one block of rows per workgroup."""
    for heads in (1, 16, 40, 128, 300, 448, 896):
        for rows in (1, 32, 33, 64, 100, 256):
            for n in (1, 300, 700, 1400, 2048):
                for room in (0, heads * n * 4, heads * n * 8 - 1, heads * n * 8, heads * n * 32):
                    got = splits(dtype, d, heads, rows, rows, n, 0, 0, room)
                    assert got in (0, 1, (rows + 31) // 32)
                    assert got <= 1 or got * heads * n * 4 <= room


def test_no_hand_written_instruction_reads_an_unfinished_result():
    if not os.path.exists(hz.HIPCC):
        pytest.skip("hipcc not present")
    kernels = [k for k in hz._kernels(hz._isa("score_rows.hip")) if any("v_mfma" in t for t, _ in k[1])]
    assert len(kernels) == 28
    for name, ins, labels in kernels:
        for producer, need in ((lambda t: "v_mfma" in t, hz.MFMA_8_PASS_WAIT_STATES),
                               (lambda t: t.startswith(("v_exp_f32", "v_log_f32", "v_rcp_f32")), hz.TRANS_WAIT_STATES)):
            assert not hz.exposed_readers(ins, labels, producer, need), name
        sgpr = hz.hand_written_sgpr_readers_behind_valu(ins, 5)
        assert not sgpr, (name, sgpr[:3])

"""How launches are cut (csrc/launch_rules.h), host code only: sizes that were timed on both sides of a rule go to the side that
was faster."""
import ctypes
import os

import pytest

from paper_2509_17396_amd import binding as ep
from paper_2509_17396_amd import build


@pytest.fixture(scope="module")
def rules():
    so = os.path.join(os.path.dirname(build.LIB), "selftest", "liblaunch_rules.so")
    if not os.path.exists(so):
        build.build_selftests()
    return ctypes.CDLL(so)


BF16, F32 = ep.DTYPE_BF16, ep.DTYPE_F32


# dtype, head_dim, rows per workgroup, heads, 64-key tiles; what pass 2 took with the fit's splits against the estimate's
@pytest.mark.parametrize("fitted,sizes", [
    (False, [(BF16, 136, 128, 32, 204), (BF16, 136, 128, 224, 16), (BF16, 192, 128, 64, 204), (BF16, 256, 128, 64, 128),  # 1.14 .. 1.32
             (F32, 72, 128, 64, 128), (F32, 96, 128, 32, 204), (F32, 128, 128, 64, 128),                                   # 1.08 .. 1.13
             (BF16, 32, 32, 896, 16), (BF16, 32, 32, 512, 40), (BF16, 8, 32, 256, 128), (F32, 64, 64, 896, 64)]),          # 1.10 .. 1.21
    (True, [(BF16, 32, 64, 64, 64), (BF16, 96, 128, 96, 16), (BF16, 128, 128, 896, 64), (BF16, 64, 256, 96, 64),            # 0.70 .. 0.88
            (BF16, 136, 32, 32, 64), (BF16, 256, 64, 96, 64), (F32, 72, 64, 32, 64), (F32, 128, 32, 64, 16),
            (BF16, 40, 32, 224, 64), (BF16, 64, 192, 96, 128)])])
def test_key_splits_of_the_max_reduction(rules, fitted, sizes):
    for size in sizes:
        a, b = ctypes.c_int(0), ctypes.c_int(0)
        assert bool(rules.max_splits(*size, ctypes.byref(a), ctypes.byref(b))) == fitted, size
        assert 1 <= a.value <= 32 and 1 <= b.value <= 32

"""The selection's cuts of the interval that holds the M-th largest score: rows that need none, one or several of them, that
fill a single part of a cut, that tie at the row's minimum (whose part is not counted), and the ends of the float order."""
import numpy as np
import pytest

from tests import parity_util as pu
from tests.test_gpu_parity import gpu_topk

pytestmark = pytest.mark.gpu


def order_keys(x):
    u = x.view(np.uint32)
    return np.where(u >> 31, ~u, u | np.uint32(1 << 31)).astype(np.uint32)


def rows_of(kind, rng, n):
    if kind == "nested":       # every cut leaves most of the row in one part
        x = 1.0 + np.ldexp(rng.integers(0, 64, n), -rng.integers(6, 23, n)).astype(np.float64)
    elif kind == "one_part":   # outliers stretch the range, everything else is within a part of it
        x = np.where(rng.random(n) < 0.01, 10.0 ** rng.uniform(-30, 30, n), 1 + rng.integers(0, 90, n) * 2.0 ** -23)
    elif kind == "minimum":    # weights that have underflowed
        x = np.where(rng.random(n) < 0.8, 0.0, rng.random(n))
    elif kind == "two":        # two values
        x = np.where(rng.random(n) < 0.5, 0.25, 0.75)
    else:                      # every bit pattern, both NaNs at the ends and the two zeros among them
        bits = rng.integers(0, 1 << 32, n, dtype=np.uint64).astype(np.uint32)
        ends = np.array([0xffffffff, 0x7fffffff, 0x80000000, 0, 0xff800000, 0x7f800000], np.uint32)
        bits[rng.integers(0, n, n // 3)] = rng.choice(ends, n // 3)
        return bits.view(np.float32)
    return x.astype(np.float32)


@pytest.mark.parametrize("kind", ["nested", "one_part", "minimum", "two", "bits"])
@pytest.mark.parametrize("n", [2, 64, 65, 66, 1000, 4096, 8200, 24576, 32768])
def test_topk_of_rows_that_need_several_cuts(n, kind):
    rng = np.random.default_rng(n)
    for m in sorted({1, n // 5 + 1, n // 2, n - 1}):
        if not 1 <= m < n:
            continue
        print(f"[gpu test] topk n={n} m={m} {kind}", flush=True)
        s = np.stack([rows_of(kind, rng, n) for _ in range(3)])[None]
        got = gpu_topk(s, m)
        pu.assert_keep_valid(got, n, m, kind)
        for h in range(3):  # largest key first, the lower index among equal ones
            want = np.sort(np.lexsort((np.arange(n), -order_keys(s[0, h]).astype(np.int64)))[:m])
            np.testing.assert_array_equal(got[0, h], want, err_msg=f"row {h}")

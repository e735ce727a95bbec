"""Errors of the scores against float64 for the rows whose normalisers are kept apart (fp32, and bf16 of any length but 64
and 128), and the most scoring rows per KV head, where their two numbers per row leave room for one query tile in LDS."""
import numpy as np
import pytest
import torch

from oracle import epicache_oracle as orc
from paper_2509_17396_amd import synth
from tests import parity_util as pu
from tests.test_gpu_parity import gpu_score

pytestmark = pytest.mark.gpu

ROWS = [("f32", 16), ("f32", 64), ("f32", 128), ("bf16", 8), ("bf16", 40), ("bf16", 96), ("bf16", 112), ("bf16", 192),
        ("bf16", 256)]


def inputs(dtype, d, hq, hkv, p, n, logits, seed):
    g = torch.Generator().manual_seed(seed)
    t = torch.float32 if dtype == "f32" else torch.bfloat16
    q = (logits * torch.randn(2, hq, p, d, generator=g)).to(t)
    return q, torch.randn(2, hkv, n, d, generator=g).to(t)


@pytest.mark.parametrize("reduce", [orc.REDUCE_MAX, orc.REDUCE_SUM], ids=["max", "sum"])
@pytest.mark.parametrize("dtype,d", ROWS)
@pytest.mark.parametrize("hq,hkv,p,n", [(2, 2, 20, 384), (8, 2, 32, 1500), (14, 2, 33, 2100), (8, 2, 70, 5000)],
                         ids=["R20", "R128", "R231", "R280"])
def test_mean_error_of_small_logits(dtype, d, hq, hkv, p, n, reduce):
    """A weight takes an exponential (2^-23 at most), a reciprocal and a product (2^-24 each) and a logit of about 0.3
    whose rounding is as small; the mean over keys is at most half of that sum, 1.2e-7, and half as much again."""
    print(f"[gpu test] precision {dtype} d={d} Hq={hq} Hkv={hkv} p={p} N={n} reduce={reduce}", flush=True)
    q, k = inputs(dtype, d, hq, hkv, p, n, 0.3, d + n)
    want = orc.score(*pu.oracle_inputs(q, k), n, reduce)
    got = gpu_score(q.cuda(), k.cuda(), n, n // 2, reduce).astype(np.float64)
    assert (np.abs(got - want) / want).mean() <= 1.8e-7


@pytest.mark.parametrize("dtype,d", ROWS)
@pytest.mark.parametrize("hq,hkv,p,n", [(8, 2, 32, 384), (4, 4, 64, 1500), (14, 2, 33, 2100)], ids=["R128", "R64", "R231"])
def test_error_of_a_key_that_holds_its_row(dtype, d, hq, hkv, p, n):
    """Logits of some 12: where one key holds more than 0.9 of a row its weight is 1 less a small sum, so neither the size
    of the logits nor how far the maximum climbed may show in it: a few roundings of 2^-24, 1.5e-7 in the mean, and a
    tenth of the error of the other weights (2^-24 of a logit of 40)."""
    print(f"[gpu test] precision, dominant keys {dtype} d={d} Hq={hq} Hkv={hkv} p={p} N={n}", flush=True)
    q, k = inputs(dtype, d, hq, hkv, p, n, 12.0, d + n)
    want = orc.score(*pu.oracle_inputs(q, k), n, orc.REDUCE_MAX)
    got = gpu_score(q.cuda(), k.cuda(), n, n // 2, orc.REDUCE_MAX).astype(np.float64)
    held = want > 0.9
    assert held.sum() >= 20
    assert (np.abs(got - want) / want)[held].mean() <= 4e-7


@pytest.mark.parametrize("reduce", [orc.REDUCE_MAX, orc.REDUCE_SUM], ids=["max", "sum"])
@pytest.mark.parametrize("dtype,d", [("bf16", 40), ("bf16", 96), ("bf16", 136), ("bf16", 256), ("f32", 64), ("f32", 128)])
@pytest.mark.parametrize("rows", [8256, 12288, 12289, 16384])
def test_most_scoring_rows(dtype, d, rows, reduce):
    print(f"[gpu test] {rows} scoring rows {dtype} d={d} reduce={reduce}", flush=True)
    q, k = inputs(dtype, d, 1, 1, rows, 193, 1.0, rows)
    want = orc.score(*pu.oracle_inputs(q, k), 193, reduce)
    pu.assert_scores_close(gpu_score(q.cuda(), k.cuda(), 193, 100, reduce), want, 1e-5, f"R={rows}")
